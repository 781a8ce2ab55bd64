// Device kernels and launch templates of the implicit-GEMM convolutions (gfx950).
// See conv.hip for the map from the three convolution calls onto these kernels.
#pragma once

#include <type_traits>

#include "common.h"

namespace pt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Raw 8 x bf16 load from base + off (elements).  VEC: one 16-byte load (off*2 is 16-byte aligned and all
// 16 bytes are readable).  Otherwise eight 2-byte loads, where element e >= nvalid re-reads element 0 so
// that nothing beyond the row's logical extent is touched.  No branches: callers clamp `off` to a
// readable location for rows that are out of range and zero the result with mask8().
template <bool VEC>
__device__ __forceinline__ uint4 ldg8(const uint16_t* __restrict__ base, uint32_t off, int nvalid) {
    if constexpr (VEC) {
        return *reinterpret_cast<const uint4*>(base + off);
    } else {
        uint32_t d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = base[off + (2 * i < nvalid ? 2 * i : 0)];
            const uint32_t hi = base[off + (2 * i + 1 < nvalid ? 2 * i + 1 : 0)];
            d[i] = lo | (hi << 16);
        }
        return make_uint4(d[0], d[1], d[2], d[3]);
    }
}

// Per-dword masks that keep elements [0, nvalid) of an 8 x bf16 vector.
struct Mask8 {
    uint32_t m[4];
};
__device__ __forceinline__ Mask8 make_mask8(int nvalid) {
    Mask8 k;
#pragma unroll
    for (int i = 0; i < 4; ++i) k.m[i] = nvalid >= 2 * i + 2 ? 0xffffffffu : (nvalid == 2 * i + 1 ? 0xffffu : 0u);
    return k;
}
__device__ __forceinline__ uint4 mask8(uint4 v, bool ok, const Mask8& k) {
    v.x = ok ? (v.x & k.m[0]) : 0u;
    v.y = ok ? (v.y & k.m[1]) : 0u;
    v.z = ok ? (v.z & k.m[2]) : 0u;
    v.w = ok ? (v.w & k.m[3]) : 0u;
    return v;
}

// LDS reads issued as inline assembly are ordered only by explicit waits: the compiler neither moves them nor
// adds waits of its own.  The result registers must not be touched before lds_wait() has been applied to them.
// Waits until at most N of this wave's LDS reads are outstanding (they return in order) and makes `first`
// depend on the wait; lds_tie() extends the dependence to further registers, also to those whose values nobody
// wants: a read in flight would overwrite whatever else the compiler had put there.
template <int N, typename V>
__device__ __forceinline__ void lds_wait(V& first) {
    static_assert(N >= 0 && N < 16, "lgkmcnt range");
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(first) : "n"(N));
}
template <typename V>
__device__ __forceinline__ void lds_tie(V& v) {
    asm volatile("" : "+v"(v));
}
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// XCD-aware block remap: hardware deals consecutive workgroup ids round-robin to the 8 XCDs; give
// each XCD a contiguous range of logical tiles so tiles that share operands share an L2.
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
    const int xcd = bid & 7, q = bid >> 3;
    const int per = nb >> 3, rem = nb & 7;
    return xcd * per + min(xcd, rem) + q;
}

// floor(m / d) for 0 <= m < 2^31 through a host-made reciprocal: with l = ceil(log2 d) and magic = ceil(2^(31 + l) / d) (at
// most 32 bits) the error magic * d - 2^(31 + l) is below 2^l, so m * magic / 2^(31 + l) is off by less than 1 / d.  No
// branch and no special divisor: a workgroup's first load waits for these divisions.
struct FastDiv {
    uint32_t d, magic, shift;
};
inline FastDiv make_fastdiv(int64_t d) {
    uint32_t l = 0;
    while ((1ll << l) < d) ++l;
    return FastDiv{(uint32_t)d, (uint32_t)(((1ull << (31 + l)) + (uint64_t)d - 1) / (uint64_t)d), l};
}
__device__ __forceinline__ uint32_t fdiv(uint32_t m, FastDiv f) { return __umulhi(2 * m, f.magic) >> f.shift; }
// The same for m * d < 2^32: one multiplication, and d == 1 apart.  In the register-staged kernels, whose pixel divisions stand
// in the step loop or in front of a short one, it is the faster form (element-wise loads, 1 x 1 calls of 5 us: 0.3 us; weight
// gradients 1 to 9 %).
struct SmallDiv {
    uint32_t d, magic;
};
inline SmallDiv make_smalldiv(int64_t d) { return SmallDiv{(uint32_t)d, d == 1 ? 0u : make_magic((uint32_t)d)}; }
__device__ __forceinline__ uint32_t fdiv(uint32_t m, SmallDiv f) { return f.d == 1 ? m : __umulhi(m, f.magic); }

// ------------------------------------------------------------------------------------------- //
// forward / input-gradient implicit GEMM
// ------------------------------------------------------------------------------------------- //
// Byte offset of grid point m = (n * gH + gi) * gW + gj in a tensor: m * point + (m / gW) * row + n * image + origin (mod 2^32).
struct RowOffsets {
    uint32_t point, row, image, origin;
};
struct IgemmArgs {
    const uint16_t* A;  // gathered activations (x or dy)
    const uint16_t* B;  // weights, [Nout][b_taps][bpitch], reduction channel innermost
    uint16_t* D;        // output activations
    int M;              // output pixels of this launch = images * gH * gW
    FastDiv gW, gH;     // output pixel grid per image (of this launch): width, height
    SmallDiv sW, sH;    // the same for the register-staged kernel (here, among the arguments that it reads first)
    int srcH, srcW, apitch;
    int h_mul, h_add, w_mul, w_add;  // source coordinate of tap (0,0) for grid point (i,j)
    int tr_step, ts_step;            // source coordinate step per tap index
    int TR, TS;                      // taps of this launch
    int Cred, CredP;                 // reduction channels, and rounded up to 8
    // Folded small-channel mode (direct kernel only): when a pixel holds fewer than 64 padded channels and
    // pixels are dense (pitch == padded channels), the S taps of a filter row are one contiguous run of
    // S*Cfold elements in both operands, so a reduction step covers several taps.  Then TS == 1,
    // Cred == CredP == S*Cfold, TSm == S taps per row in the validity mask, Creal real channels per tap.
    int fold, TSm, Creal;
    FastDiv Cfold;
    int b_tap0, b_tr_stride, b_ts_stride, b_taps;
    int bpitch, Nout;
    int DH, DW, d_hmul, d_hadd, d_wmul, d_wadd, dpitch;  // destination pixel = (i*d_hmul+d_hadd, j*d_wmul+d_wadd)
    int d_linear;                                        // destination pixel index == m
    int nk;                                              // reduction steps of BK
    int tiles_n;
    int d_vec;    // 8-byte stores allowed (pitch % 4 == 0, base 8-byte aligned)
    int d_vec16;  // 16-byte stores allowed (pitch % 8 == 0, base 16-byte aligned)
    // Direct kernel, channel counts that are not multiples of 8: which of the eight 16-byte chunks of a 64-channel block
    // end in undefined padding elements.  Byte b of tail_kv = chunk bits of block b of a folded run; otherwise byte 0
    // describes the last block of a tap (the only one with a tail) and byte 7 is zero.
    uint64_t tail_kv;
    int tail_nvalid;  // defined elements of a tail chunk (1..7), 8 when there is none
    int pad_zero;     // the caller vouches that the padding channels of both operands hold zeros
    // Input gradient of a strided layer whose only stride-parity class with filter taps is (0, 0): every destination
    // pixel lies in the zf_h x zf_w cell anchored at one pixel of that class, and the launch clears the rest of each
    // cell itself (1 x 1 = off).  Direct kernel, 16-byte stores only.
    int zf_h, zf_w;
    // STATS instantiations (forward only): per-channel sums of the stored (bf16-rounded) outputs and of their
    // squares over the tile's valid pixels, one row per pixel tile: stats[(q * tiles_m + tile_m) * Nout + channel],
    // q = 0 sums, q = 1 sums of squares - the layout the normalisation's finish pass reads.
    float* stats;
    int tiles_m;
    // Direct kernel, buffer addressing of the gathered operand: a row's offset plus a_guard is non-negative for
    // every row, a reduction step's offset minus a_smin is non-negative for every step (both in elements; the
    // buffer's base address absorbs the two shifts).  a_all_valid: no tap of any row ever leaves the source image.
    int a_guard, a_smin, a_all_valid;
    // Direct kernel: the raised wave priority of the reduction loop also outside it.  Off for a launch that runs alone; the
    // input gradient, which is meant to run beside weight gradients of other layers, keeps its set-up and its stores
    // ahead of them too.
    int edge_prio;
    int grid_x;  // direct kernel: workgroups (tiles) of this problem inside a launch that may hold several problems
    int m_fast;  // small tiles: consecutive tiles run along the pixels (and share weights), not along the outputs
    // Direct kernels: the above, ready for use in a workgroup's set-up (make_igemm_offsets).
    FastDiv t_div;  // tiles along the axis that consecutive tiles run along
    RowOffsets src, dst;
    int ch_mul, ch_add, cw_mul, cw_add;  // taps inside the source image: rows [gi * ch_mul + ch_add, + srcH), columns alike
    uint64_t tap_rep;                    // bit r * TSm for every filter row r
};

// The direct kernel takes up to four problems per launch, one per blockIdx.y (the stride-parity classes of a strided
// input gradient: disjoint output pixels, the same operands): workgroups past a problem's own tile count leave at once.
constexpr int kIgemmMaxProblems = 4;
struct IgemmArgsN {
    IgemmArgs a[kIgemmMaxProblems];
};

// Fills tail_kv / tail_nvalid (see IgemmArgs) for the direct kernel's 64-channel blocks.
inline void set_tail_tables(IgemmArgs& a) {
    a.tail_kv = 0;
    a.tail_nvalid = 8;
    const int creal = a.fold ? a.Creal : a.Cred;
    if ((creal & 7) == 0) return;
    a.tail_nvalid = creal & 7;
    const int tail_chunk = creal >> 3;  // chunk index of the tail inside one run
    if (!a.fold) {
        a.tail_kv = 1ull << (tail_chunk & 7);  // in the last block of the tap
        return;
    }
    const int per = (int)(a.Cfold.d >> 3);  // chunks per run
    const int nblk = (a.CredP + 63) >> 6;   // <= 8: igemm_fold sees to it
    for (int c = 0; c < nblk * 8; ++c)
        if (c % per == tail_chunk) a.tail_kv |= 1ull << c;
}

// VEC: every operand row is 16-byte aligned (pitches are multiples of 8 elements).
template <int BM, int BN, int BK, int WGM, int WGN, int STAGES, int MINB, bool VEC>
__global__ __launch_bounds__(64 * WGM * WGN, MINB) void k_igemm(const IgemmArgs a) {
    constexpr int NT = 64 * WGM * WGN;
    constexpr int LDK = BK + 8;  // LDS row pitch in elements (16-byte pad: conflict-free 16-byte reads)
    constexpr int KV = BK / 8;
    constexpr int RPP = NT / KV;
    constexpr int AP = BM / RPP, BP = BN / RPP;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    constexpr int STAGE_ELEMS = (BM + BN) * LDK;
    static_assert(AP >= 1 && BP >= 1 && TM >= 1 && TN >= 1 && BM % RPP == 0 && BN % RPP == 0, "tile config");
    static_assert(STAGES == 1 || STAGES == 2, "stages");
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int n0 = (tile % a.tiles_n) * BN;
    const int m0 = (tile / a.tiles_n) * BM;

    // ---- loader state -------------------------------------------------------------------------
    const int kv = tid % KV, lrow = tid / KV;
    int c0 = kv * 8, tr = 0, ts = 0;
    while (c0 >= a.CredP) {
        c0 -= a.CredP;
        if (++ts == a.TS) { ts = 0; ++tr; }
    }
    int a_hw[AP];    // (h0 << 16) | (w0 & 0xffff): source coordinate of tap (0,0)
    int a_poff[AP];  // linear source pixel of tap (0,0)
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int m = m0 + lrow + i * RPP;
        int h0 = -30000, w0 = 0, poff = 0;
        if (m < a.M) {
            const uint32_t row = fdiv((uint32_t)m, a.sW), gj = m - row * a.sW.d;
            const uint32_t n = fdiv(row, a.sH), gi = row - n * a.sH.d;
            h0 = (int)gi * a.h_mul + a.h_add;
            w0 = (int)gj * a.w_mul + a.w_add;
            poff = ((int)n * a.srcH + h0) * a.srcW + w0;
        }
        a_hw[i] = (h0 << 16) | (w0 & 0xffff);
        a_poff[i] = poff;
    }
    const uint32_t b_rowlen = (uint32_t)a.b_taps * a.bpitch;

    uint4 ra[AP], rb[BP];
    bool oka[AP], okb[BP];
    Mask8 kmask;
    // issue the global loads of the next reduction step (raw, unmasked)
    auto gload = [&]() {
        const bool kok = tr < a.TR;
        const int nvalid = kok ? a.Cred - c0 : 0;
        kmask = make_mask8(nvalid);
        const int dh = tr * a.tr_step, dw = ts * a.ts_step;
        const int dpix = dh * a.srcW + dw;
#pragma unroll
        for (int i = 0; i < AP; ++i) {
            const int ih = (a_hw[i] >> 16) + dh, iw = (int)(short)(a_hw[i] & 0xffff) + dw;
            oka[i] = kok && (unsigned)ih < (unsigned)a.srcH && (unsigned)iw < (unsigned)a.srcW;
            const uint32_t off = (uint32_t)(a_poff[i] + dpix) * (uint32_t)a.apitch + (uint32_t)c0;
            ra[i] = ldg8<VEC>(a.A, oka[i] ? off : 0u, nvalid);
        }
        const uint32_t tapoff = (uint32_t)(a.b_tap0 + tr * a.b_tr_stride + ts * a.b_ts_stride) * (uint32_t)a.bpitch + c0;
#pragma unroll
        for (int j = 0; j < BP; ++j) {
            const int nrow = n0 + lrow + j * RPP;
            okb[j] = kok && nrow < a.Nout;
            rb[j] = ldg8<VEC>(a.B, okb[j] ? (uint32_t)nrow * b_rowlen + tapoff : 0u, nvalid);
        }
        c0 += BK;
        while (c0 >= a.CredP && tr < a.TR) {
            c0 -= a.CredP;
            if (++ts == a.TS) { ts = 0; ++tr; }
        }
    };
    auto sstore = [&](int buf) {
        uint16_t* sA = smem + buf * STAGE_ELEMS;
        uint16_t* sB = sA + BM * LDK;
#pragma unroll
        for (int i = 0; i < AP; ++i)
            *reinterpret_cast<uint4*>(&sA[(lrow + i * RPP) * LDK + kv * 8]) = mask8(ra[i], oka[i], kmask);
#pragma unroll
        for (int j = 0; j < BP; ++j)
            *reinterpret_cast<uint4*>(&sB[(lrow + j * RPP) * LDK + kv * 8]) = mask8(rb[j], okb[j], kmask);
    };

    // ---- MFMA state ---------------------------------------------------------------------------
    const int wm = wave % WGM, wn = wave / WGM;
    const int l32 = lane & 31, lk = (lane >> 5) * 8;
    f32x16 acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tn][tm][v] = 0.f;
    bool n_live[TN], m_live[TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) n_live[tn] = n0 + wn * WTN + tn * 32 < a.Nout;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) m_live[tm] = m0 + wm * WTM + tm * 32 < a.M;

    bool all_live = true;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) all_live = all_live && n_live[tn];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) all_live = all_live && m_live[tm];

    // CHECK = false: every 32x32 block of this wave is inside the output (no per-block tests)
    auto compute = [&](int buf, auto check_tag) {
        constexpr bool CHECK = decltype(check_tag)::value;
        const uint16_t* sA = smem + buf * STAGE_ELEMS;
        const uint16_t* sB = sA + BM * LDK;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 fw[TN], fp[TM];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                fw[tn] = *reinterpret_cast<const bf16x8*>(&sB[(wn * WTN + tn * 32 + l32) * LDK + ks * 16 + lk]);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
                fp[tm] = *reinterpret_cast<const bf16x8*>(&sA[(wm * WTM + tm * 32 + l32) * LDK + ks * 16 + lk]);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
                    if (!CHECK || (n_live[tn] && m_live[tm]))
                        acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[tn], fp[tm], acc[tn][tm], 0, 0, 0);
        }
    };
    // software pipeline over the reduction steps; the tile-edge test is hoisted out of the loop
    auto main_loop = [&](auto check_tag) {
        if constexpr (STAGES == 2) {
            for (int kt = 0; kt < a.nk; ++kt) {
                const int buf = kt & 1;
                if (kt + 1 < a.nk) gload();
                compute(buf, check_tag);
                if (kt + 1 < a.nk) sstore(buf ^ 1);
                __syncthreads();
            }
        } else {
            for (int kt = 0; kt < a.nk; ++kt) {
                if (kt + 1 < a.nk) gload();
                compute(0, check_tag);
                __syncthreads();
                if (kt + 1 < a.nk) {
                    sstore(0);
                    __syncthreads();
                }
            }
        }
    };
    gload();
    sstore(0);
    __syncthreads();
    if (all_live) main_loop(std::false_type{});
    else main_loop(std::true_type{});

    // ---- epilogue: lane holds pixel (column) l32, channels 8g + 4*(lane/32) + {0..3} of each block --
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int m = m0 + wm * WTM + tm * 32 + l32;
        if (m >= a.M) continue;
        int64_t dpix;
        if (a.d_linear) {
            dpix = (int64_t)m * a.dpitch;
        } else {
            const uint32_t row = fdiv((uint32_t)m, a.sW), gj = m - row * a.sW.d;
            const uint32_t n = fdiv(row, a.sH), gi = row - n * a.sH.d;
            dpix = (((int64_t)n * a.DH + (int)gi * a.d_hmul + a.d_hadd) * a.DW + (int)gj * a.d_wmul + a.d_wadd) * a.dpitch;
        }
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int ch = n0 + wn * WTN + tn * 32 + 8 * g + (lane >> 5) * 4;
                if (ch >= a.Nout) continue;
                const float v0 = acc[tn][tm][4 * g + 0], v1 = acc[tn][tm][4 * g + 1];
                const float v2 = acc[tn][tm][4 * g + 2], v3 = acc[tn][tm][4 * g + 3];
                uint16_t* dst = a.D + dpix + ch;
                if (a.d_vec && ch + 3 < a.Nout) {
                    uint2 o;
                    o.x = pack_bf16x2(v0, v1);
                    o.y = pack_bf16x2(v2, v3);
                    *reinterpret_cast<uint2*>(dst) = o;
                } else {
                    dst[0] = f32_to_bf16(v0);
                    if (ch + 1 < a.Nout) dst[1] = f32_to_bf16(v1);
                    if (ch + 2 < a.Nout) dst[2] = f32_to_bf16(v2);
                    if (ch + 3 < a.Nout) dst[3] = f32_to_bf16(v3);
                }
            }
        }
    }
}

template <int BM, int BN, int BK, int WGM, int WGN, int STAGES, int MINB, bool VEC = true>
inline hipError_t launch_igemm_cfg(IgemmArgs& a, hipStream_t st) {
    constexpr int NT = 64 * WGM * WGN;
    constexpr size_t lds = (size_t)STAGES * (BM + BN) * (BK + 8) * 2;
    auto kern = k_igemm<BM, BN, BK, WGM, WGN, STAGES, MINB, VEC>;
    static LdsOptIn opt_in;
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void*>(kern), lds); e != hipSuccess) return e;
    const int tiles_m = (int)ceil_div(a.M, BM);
    a.tiles_n = (int)ceil_div(a.Nout, BN);
    a.nk = (int)ceil_div((int64_t)a.TR * a.TS * a.CredP, BK);
    hipLaunchKernelGGL(kern, dim3(tiles_m * a.tiles_n), dim3(NT), lds, st, a);
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------- //
// forward / input-gradient implicit GEMM with direct global->LDS loads (vector path)
// ------------------------------------------------------------------------------------------- //
// Same problem mapping as k_igemm, different data movement: 16-byte loads land in LDS without
// passing through registers (buffer_load_dwordx4 ... lds), so several reduction steps can be in flight
// per workgroup at no register cost.  A wave-level load fills 1 KiB of LDS contiguously (lane l ->
// bytes [16l, 16l+16)), i.e. 8 tile rows of BK = 64 elements; rows are unpadded and the eight 16-byte
// chunks of a row are XOR-swizzled with ((row >> 1) & 7) so that the MFMA operand reads (16 consecutive
// rows, same logical chunk) fall into 16 different bank groups.  The swizzle is applied on the global
// side: the lane that owns physical chunk p of a row fetches logical chunk p ^ swz(row).
// Taps outside the image and chunks past the channel count are fetched as zeros (an out-of-range buffer offset, see
// the kernel).  RAGGED = the channel count is not a multiple of 64 (the last block of a run is partly zeros); TAIL = in
// addition some 8-chunk ends in undefined padding elements, which are cleared in LDS before the stage is published.
// The 16-byte zero page below serves the weight-gradient kernel's general gather, which still uses per-lane addresses.
__device__ __attribute__((aligned(16))) uint32_t g_zero16[4] = {0u, 0u, 0u, 0u};

typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(1))) void* glb_void_ptr;

// Workgroup barrier without the memory fence of __syncthreads(): the fence would wait for every
// outstanding global->LDS load, which is exactly what the software pipeline must not do.  Callers
// wait explicitly (vmcnt for landed DMA data, lgkmcnt for their own LDS writes) before calling.
__device__ __forceinline__ void barrier_nofence() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Per-lane choice between two global addresses, kept opaque so that it stays one load instruction.
__device__ __forceinline__ glb_void_ptr pick_ptr(bool ok, const uint16_t* p, const uint16_t* z) {
    uint64_t v = ok ? (uint64_t)(uintptr_t)p : (uint64_t)(uintptr_t)z;
    asm volatile("" : "+v"(v));
    return (glb_void_ptr)(uintptr_t)v;
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    // s_waitcnt immediate: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14 ; only vmcnt constrained
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// The same, and until this wave's LDS reads have returned.
template <int N>
__device__ __forceinline__ void wait_vmcnt_lds() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

__device__ __forceinline__ uint32_t swap_lane_pair(uint32_t v) {  // lanes 2i and 2i + 1 trade values
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true);
}
// The taps of grid point (gi, gj) that read outside the source image: a bit r * TSm + s each, set (bits past the last tap
// too).  The taps inside are an interval of filter rows times an interval of columns: the column bits, repeated in every
// row by a multiplication, cut to the rows' bits.
struct TapSkip {
    int lo, hi;
};
__device__ __forceinline__ TapSkip tap_skip(const IgemmArgs& a, int gi, int gj) {
    const int r = gi * a.ch_mul + a.ch_add, s = gj * a.cw_mul + a.cw_add;
    const int r0 = min(max(r, 0), a.TR) * a.TSm, r1 = min(max(r + a.srcH, 0), a.TR) * a.TSm;
    const int s0 = min(max(s, 0), a.TSm), s1 = min(max(s + a.srcW, 0), a.TSm);
    if (a.TR * a.TSm < 32)  // uniform
        return {(int)~(((1u << s1) - (1u << s0)) * (uint32_t)a.tap_rep & ((1u << r1) - (1u << r0))), -1};
    auto below = [](int n) { return n > 63 ? ~0ull : (1ull << n) - 1; };
    const uint64_t valid = (below(s1) & ~below(s0)) * a.tap_rep & (below(r1) & ~below(r0));
    return {(int)~(uint32_t)valid, (int)~(uint32_t)(valid >> 32)};
}

// DEEP = a step's fragments are read into registers during the step before it.  Its LDS is then free for the loads of step
// STAGES later from the step's own barrier on, a stage earlier than otherwise, and no MFMA waits for the LDS behind a barrier.
// For reductions long enough to pay for the first reads, on launches of about one workgroup per CU (pick_igemm_deep).
// With three stages every step but the last ones sends out a later step's loads between its MFMAs, a quarter with each 16
// channels (with two they go out ahead of the step's reads, see main_loop): the 64 or more load instructions of a workgroup
// take the CU's address unit 16 clocks each, and ahead of the fragment reads they held those, and the MFMAs, back for half
// a step.  Forward, 3 x 3, batch 64, operands from memory / in the caches: 128 x 64 tiles, 7 x 7 512 -> 512 29.4 / 28.1 ->
// 28.1 / 23.6 us; deep, 128 x 128 tiles in three stages, 14 x 14 256 -> 256 23.9 / 21.8 -> 20.3 / 17.6 us (MFMAs alone,
// without loads and reads: 12.2), 1 x 1 1024 -> 256 16.7 / 11.1 -> 13.5 / 9.7; deep, 256 x 128, 28 x 28 128 -> 128 20.3 /
// 18.1 -> 19.3 / 17.3.  Bound now by fragment reads and MFMAs, which with one barrier a step overlap to 0.31 us of a 128 x
// 128 x 64 step (MFMAs alone 0.23), and on 128 x 64 tiles by the operands from the L2 (20 TB/s).
// TAIL = some run of channels ends inside an 8-chunk whose remaining elements are undefined.
// STATS = also reduce the stored outputs to per-channel sums and sums of squares (see IgemmArgs::stats).
// AV = the caller has established that every tap of every row lies inside the source image (no validity tests).
// FOLD = the problem may be a folded one (without AV; with a branch for it in the loop the loads no longer share a block with
// the step's LDS reads and MFMAs: 22.8 instead of 22.2 us on 14 x 14 x 256 -> 256, 3 x 3, batch 64).
template <int BM, int BN, int WGM, int WGN, int STAGES, bool RAGGED, bool TAIL, bool STATS, bool AV, bool FOLD, bool DEEP>
__global__ __launch_bounds__(64 * WGM * WGN, 1) void k_igemm_dl(const IgemmArgsN problems) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
    const IgemmArgs a = problems.a[blockIdx.y];  // (a copy: the fields then live in scalar registers as kernel arguments do)
    if (a.edge_prio) __builtin_amdgcn_s_setprio(2);
    constexpr int NW = WGM * WGN, BK = 64;
    constexpr int GA = BM / 8, GB = BN / 8;    // 8-row groups = wave-level loads per stage
    constexpr int LA = GA / NW, LB = GB / NW;  // loads per lane per stage
    constexpr int LPT = LA + LB;
    constexpr int STAGE_BYTES = (BM + BN) * 128;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    static_assert(NW % 2 == 0 && GA % NW == 0 && GB % NW == 0 && LA >= 1 && LB >= 1 && TM >= 1 && TN >= 1, "tile config");
    static_assert(STAGES >= 2 && (STAGES - 1) * LPT < 64 && !(DEEP && (TAIL || STATS || FOLD)), "stages");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_b[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = xcd_remap(blockIdx.x, a.grid_x);
    const int tile_m = (int)fdiv((uint32_t)tile, a.t_div);
    const int n0 = (tile - tile_m * a.tiles_n) * BN, m0 = tile_m * BM;

    // A reduction step is (filter tap, block of 64 reduction channels): the same for every lane, so the
    // tap offsets and the channel base live in scalar registers.
    const int lrow = lane >> 3;                                      // row inside an 8-row group
    const int kv = (lane & 7) ^ ((((wave & 1) << 2) | (lane >> 4)));  // logical 8-element chunk this lane fetches
    const int kvoff = kv * 8;

    // per-lane row constants: byte offset of tap (0,0) + chunk, and a bit per tap: tap outside the image.
    // Rows past the end of the problem are clamped to the last row: their results are never stored.
    // A workgroup waits for all of this before its first load (two WGs of eight waves on a CU: about 3 ns an instruction),
    // so what does not depend on the lane is made on the host and nothing here branches or loops: 28 x 28 x 128 -> 128,
    // 3 x 3, batch 64: 1.4 us from a workgroup's start to its first load with a loop over the taps and divisions.
    uint32_t a_v[LA], b_v[LB];
    int skip_lo[LA], skip_hi[LA];  // bit r * TSm + s: tap (r, s) of this row lies outside the image (hi: from the 33rd tap on)
#pragma unroll
    for (int j = 0; j < LA; ++j) {
        const uint32_t m = (uint32_t)min(m0 + (wave + NW * j) * 8 + lrow, a.M - 1);
        const uint32_t row = fdiv(m, a.gW), n = fdiv(row, a.gH);
        a_v[j] = m * a.src.point + row * a.src.row + n * a.src.image + a.src.origin + (uint32_t)kvoff * 2u;
        if constexpr (!AV) {
            const TapSkip t = tap_skip(a, (int)(row - n * a.gH.d), (int)(m - row * a.gW.d));
            skip_lo[j] = t.lo;
            skip_hi[j] = t.hi;
        }
    }
    const uint32_t b_rowbytes = (uint32_t)a.b_taps * a.bpitch * 2u;
#pragma unroll
    for (int j = 0; j < LB; ++j)
        b_v[j] = (uint32_t)min(n0 + (wave + NW * j) * 8 + lrow, a.Nout - 1) * b_rowbytes + (uint32_t)kvoff * 2u;
    if (blockIdx.x >= (unsigned)a.grid_x) return;  // the whole workgroup: the launch is as wide as its largest problem
    // Both operands are fetched with buffer loads: the per-lane part of an address (row, 8-element chunk) is a
    // constant byte offset (voffset), the part that changes from step to step (filter tap, channel block) is the same
    // for every lane and travels in a scalar register (soffset), and a lane that must read zeros (tap outside the
    // image, chunk past the channel count) passes an out-of-range voffset, for which the load writes zeros to LDS.
    // The reduction loop is bound by the number of instructions a wave issues, so a step costs no vector arithmetic
    // beyond those validity tests.  The base address of the gathered operand is shifted so that both parts are
    // non-negative (it may point outside the tensor: only valid taps are ever fetched).
    constexpr uint32_t kBufRecords = 0xffffff00u, kBufOut = 0xffffffffu, kBufFlags = 0x00020000u;
    const __amdgpu_buffer_rsrc_t a_srd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(a.A) + ((int64_t)a.a_smin - a.a_guard), 0, kBufRecords, kBufFlags);
    const __amdgpu_buffer_rsrc_t b_srd = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.B), 0, kBufRecords, kBufFlags);

    // With taps outside the image the next step to issue is kept as running scalar offsets, to which a step adds 64 channels and,
    // behind a branch at the end of a tap's last step, a constant (next filter column, next filter row); which lanes read zeros,
    // which changes with the tap only, is worked out there too.  14 x 14 x 256 -> 256, 3 x 3, batch 64: 22.8 us; both recomputed in
    // every step 23.1, the test alone in every step 24.0; selects instead of the branch 0 to 2 % slower.  With none outside (mostly
    // 1 x 1 layers of few steps) there is no test, and what the constants take ahead of the first load is not won back: 28 x 28 x
    // 512 -> 128 12.96 us with them, 12.70 with the offsets from tap and block.
    const int nblk = (a.CredP + BK - 1) / BK;
    const int ts_a = a.ts_step * a.apitch * 2, ts_b = a.b_ts_stride * a.bpitch * 2, back = (nblk - 1) * BK * 2;
    const int col_a = ts_a - back, col_b = ts_b - back;
    const int row_a = a.tr_step * a.srcW * a.apitch * 2 - (a.TS - 1) * ts_a - back;
    const int row_b = a.b_tr_stride * a.bpitch * 2 - (a.TS - 1) * ts_b - back;
    uint32_t s_a = (uint32_t)(-a.a_smin * 2), s_b = (uint32_t)(a.b_tap0 * a.bpitch * 2);
    int blk = nblk, col = a.TS;          // blocks left of this tap, columns left of this filter row
    int tap = 0, f_cb = 0;               // tap (folded mode: the first one of its filter row) and channel base
    int i_tr = 0, i_ts = 0, i_cb = 0;    // AV: tap and channel base
    int c_cb = 0;                        // channel base of the next step to compute (uniform)
    const uint32_t past = RAGGED && (nblk - 1) * BK + kvoff >= a.Cred ? kBufOut : 0u;  // in a tap's last block
    uint32_t a_now[LA];                  // a_v, or kBufOut in lanes that read zeros: the tap's bit sign-extended, and an OR
    auto set_tap = [&](int t) {
#pragma unroll
        for (int j = 0; j < LA; ++j)
            a_now[j] = AV ? a_v[j] : a_v[j] | (uint32_t)__builtin_amdgcn_sbfe(t & 32 ? skip_hi[j] : skip_lo[j], t & 31, 1);
    };
    set_tap(0);

    // Loads number j with j * parts / LPT == part of the next step to issue, into LDS at byte `at`; the last part moves on to
    // the step after it.
    auto issue_part = [&](uint32_t at, int part, int parts) {
        uint8_t* sbase = smem_b + at;
        uint32_t sa, sb;
        bool last;
        if constexpr (AV) {
            sa = (uint32_t)(((i_tr * a.tr_step * a.srcW + i_ts * a.ts_step) * a.apitch + i_cb - a.a_smin) * 2);
            sb = (uint32_t)(((a.b_tap0 + i_tr * a.b_tr_stride + i_ts * a.b_ts_stride) * a.bpitch + i_cb) * 2);
            last = i_cb + BK >= a.CredP;
        } else {
            sa = s_a;
            sb = s_b;
            last = blk == 1;
            // (uniform) folded: the tap depends on the lane's chunk; past the last chunk it means nothing
            if constexpr (FOLD) {
                if (a.fold && part == 0) set_tap(tap + (int)fdiv((uint32_t)(f_cb + kvoff), a.Cfold));
            }
        }
        const uint32_t zero = RAGGED ? past & (last ? ~0u : 0u) : 0u;
        static_for<0, LPT>([&](auto j_c) {
            constexpr int J = decltype(j_c)::value;
            if (J * parts / LPT != part) return;
            if constexpr (J < LA)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(a_srd, (lds_void_ptr)(sbase + (wave + NW * J) * 1024), 16, a_now[J] | zero, sa, 0, 0);
            else
                __builtin_amdgcn_raw_ptr_buffer_load_lds(b_srd, (lds_void_ptr)(sbase + BM * 128 + (wave + NW * (J - LA)) * 1024), 16,
                                                         b_v[J - LA] | zero, sb, 0, 0);
        });
        if (part != parts - 1) return;
        if constexpr (AV) {
            i_cb += BK;
            if (i_cb >= a.CredP) {
                i_cb = 0;
                if (++i_ts == a.TS) { i_ts = 0; ++i_tr; }
            }
        } else {
            if (last) {
                const bool last_col = col == 1;
                s_a += (uint32_t)(last_col ? row_a : col_a);
                s_b += (uint32_t)(last_col ? row_b : col_b);
                blk = nblk;
                col = last_col ? a.TS : col - 1;
                tap += FOLD && a.fold ? a.TSm : 1;
                f_cb = 0;
                set_tap(tap);
            } else {
                s_a += BK * 2;
                s_b += BK * 2;
                --blk;
                f_cb += BK;
            }
        }
    };
    // ---- MFMA state ---------------------------------------------------------------------------
    const int wm = wave % WGM, wn = wave / WGM;
    const int l32 = lane & 31;
    const int swz = (l32 >> 1) & 7;  // all operand rows of this lane are l32 (mod 32)
    const int kc0 = lane >> 5;
    f32x16 acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tn][tm][v] = 0.f;
    bool n_live[TN], m_live[TM];
    bool all_live = true;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        n_live[tn] = n0 + wn * WTN + tn * 32 < a.Nout;
        all_live = all_live && n_live[tn];
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        m_live[tm] = m0 + wm * WTM + tm * 32 < a.M;
        all_live = all_live && m_live[tm];
    }

    // A step = BK / 16 sub-steps of (MFMAs, fragment reads, a part of a later step's loads).
    constexpr int NF = DEEP ? 4 : 2;  // sub-steps whose fragments are in registers
    bf16x8 fw[NF][TN], fp[NF][TM];
    auto read_frags = [&](uint32_t at, int ks, int b) {
        const uint32_t pc = (uint32_t)(((ks * 2 + kc0) ^ swz) << 4);
        const uint8_t* sA = smem_b + (at + (uint32_t)(wm * WTM + l32) * 128u + pc);
        const uint8_t* sB = smem_b + (at + (uint32_t)(BM + wn * WTN + l32) * 128u + pc);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) fw[b][tn] = *reinterpret_cast<const bf16x8*>(sB + tn * 4096);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) fp[b][tm] = *reinterpret_cast<const bf16x8*>(sA + tm * 4096);
    };
    auto step = [&](uint32_t at, uint32_t next, uint32_t to, auto issue_tag, auto check_tag) {
        constexpr bool CHECK = decltype(check_tag)::value, ISSUE = decltype(issue_tag)::value;
        if constexpr (!DEEP) {
            read_frags(at, 0, 0);
            read_frags(at, 1, 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<0, 4>([&](auto ks_c) {
            constexpr int KS = decltype(ks_c)::value, F = KS % NF;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
                    if (!CHECK || (n_live[tn] && m_live[tm]))
                        acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[F][tn], fp[F][tm], acc[tn][tm], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (DEEP) read_frags(next, KS, KS);
            else if constexpr (KS < 2) read_frags(at, KS + 2, KS);
            if constexpr (ISSUE) issue_part(to, KS, 4);
            __builtin_amdgcn_sched_barrier(0);
        });
        c_cb += BK;
        if (c_cb >= a.CredP) c_cb = 0;
    };

    auto compute = [&](uint32_t at, auto check_tag) {
        constexpr bool CHECK = decltype(check_tag)::value;
        read_frags(at, 0, 0);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            if (ks + 1 < BK / 16) read_frags(at, ks + 1, (ks + 1) & 1);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
                    if (!CHECK || (n_live[tn] && m_live[tm]))
                        acc[tn][tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[ks & 1][tn], fp[ks & 1][tm], acc[tn][tm], 0, 0, 0);
        }
        c_cb += BK;
        if (c_cb >= a.CredP) c_cb = 0;
    };

    // TAIL: a channel count that is not a multiple of 8 leaves undefined elements (memory padding) at the end of the
    // last 8-chunk of every run of channels, in both operands.  The lane that fetched such a chunk overwrites them
    // with zeros in LDS once its loads have landed (writes only: nothing is read back) and before the barrier that
    // publishes the stage.  Which chunks of the current block have a tail comes from a table in the arguments.
    auto clear_tails = [&](uint32_t at) {
        asm volatile("" ::: "memory");  // keep the stores below behind the wait for the landed loads
        const int slot = a.fold ? (c_cb >> 6) : (c_cb + BK > a.Cred ? 0 : 7);
        const uint32_t bits = (uint32_t)(a.tail_kv >> (slot * 8)) & 0xffu;
        if (bits == 0) return;  // wave-uniform
        if ((bits >> kv) & 1u) {
            const int n = a.tail_nvalid;  // uniform, 1..7: bytes [2n, 16) of the chunk are cleared with <= 3 stores
            uint8_t* mine = smem_b + at + wave * 1024 + lane * 16;
#pragma unroll
            for (int j = 0; j < LA + LB; ++j) {
                uint8_t* p = mine + (j < LA ? NW * j * 1024 : BM * 128 + NW * (j - LA) * 1024);
                int e = n;
                if (e & 1) {
                    *reinterpret_cast<uint16_t*>(p + 2 * e) = 0;
                    ++e;
                }
                if (e & 2) {
                    *reinterpret_cast<uint32_t*>(p + 2 * e) = 0u;
                    e += 2;
                }
                if (e == 4) *reinterpret_cast<uint64_t*>(p + 8) = 0ull;
            }
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the clears are in LDS before the barrier
    };

    const int nk = a.nk;
    auto main_loop = [&](auto check_tag) {
        auto after = [](uint32_t v) { return v == (STAGES - 1) * STAGE_BYTES ? 0u : v + STAGE_BYTES; };
        int kt = 0;
        if constexpr (DEEP) {
            uint32_t at = 0;  // LDS of the step computed
            wait_vmcnt<(STAGES - 1) * LPT>();  // (there are at least STAGES steps)
            barrier_nofence();
            static_for<0, 4>([&](auto ks_c) { read_frags(0, decltype(ks_c)::value, decltype(ks_c)::value); });
            for (; kt + STAGES < nk; ++kt) {
                wait_vmcnt_lds<(STAGES - 2) * LPT>();
                barrier_nofence();
                step(at, after(at), at, std::true_type{}, check_tag);
                at = after(at);
            }
            for (; kt < nk; ++kt) {
                if (kt + STAGES - 1 < nk) wait_vmcnt_lds<(STAGES - 2) * LPT>();
                else wait_vmcnt_lds<0>();
                barrier_nofence();
                step(at, after(at), at, std::false_type{}, check_tag);
                at = after(at);
            }
        } else {
            // Whole rounds of the stages with nothing to test, and the last steps one by one.  With two stages the loads of the
            // next step go out ahead of this one's reads: they have only this step to arrive in.
            for (; STAGES >= 3 && kt + 2 * STAGES - 2 < nk; kt += STAGES) {
                static_for<0, STAGES>([&](auto s_c) {
                    constexpr uint32_t S = decltype(s_c)::value;
                    wait_vmcnt<(STAGES - 2) * LPT>();
                    if constexpr (TAIL) clear_tails(S * STAGE_BYTES);
                    barrier_nofence();  // stage s complete for every wave; stage (s-1) free again
                    step(S * STAGE_BYTES, 0, (S + STAGES - 1) % STAGES * STAGE_BYTES, std::true_type{}, check_tag);
                });
            }
            for (; kt < nk; kt += STAGES) {
                static_for<0, STAGES>([&](auto s_c) {
                    constexpr uint32_t S = decltype(s_c)::value;
                    const int k = kt + (int)S;
                    if (k < nk) {
                        // loads of steps k+1 .. k+STAGES-2 may stay in flight; near the end just drain
                        if (k + STAGES - 2 < nk) wait_vmcnt<(STAGES - 2) * LPT>();
                        else wait_vmcnt<0>();
                        if constexpr (TAIL) clear_tails(S * STAGE_BYTES);
                        barrier_nofence();
                        if (k + STAGES - 1 < nk) issue_part((S + STAGES - 1) % STAGES * STAGE_BYTES, 0, 1);
                        compute(S * STAGE_BYTES, check_tag);
                    }
                });
            }
        }
    };
#pragma unroll
    for (int s = 0; s < (DEEP ? STAGES : STAGES - 1); ++s)
        if (DEEP || s < nk) issue_part(s * STAGE_BYTES, 0, 1);
    // waves inside the reduction loop go first at the CU's issue arbiter: ahead of a co-resident workgroup's set-up
    // or stores, and ahead of weight-gradient waves sharing the CU from another stream (+0.4 % on the step)
    __builtin_amdgcn_s_setprio(2);
    if (all_live) main_loop(std::false_type{});
    else main_loop(std::true_type{});
    if (!a.edge_prio) __builtin_amdgcn_s_setprio(0);

    // ---- epilogue: registers -> global.  A lane holds, per 32x32 block, channels 8g + 4*(lane/32) + {0..3}
    // (g = 0..3) of pixel lane%32.  Swapping the upper half-wave of the g-even registers with the lower
    // half-wave of the g-odd ones leaves every lane with two runs of 8 consecutive channels (16 bytes of bf16).
    // Plain launches (16-byte stores, nothing else to write, every chunk a vector) first trade chunks between
    // neighbouring lanes: lane pair (2i, 2i+1) holds chunks (g-pair 0, g-pair 1) of pixels 2i and 2i+1; after the
    // exchange the even lane's pixel is written by both lanes in the first store and the odd lane's in the second,
    // so one store instruction covers 64 contiguous bytes of 16 pixels instead of 32 bytes of 32 pixels (half as
    // many partial-line write requests; a store-only probe of the two patterns differs by 15-25 %).
    const bool pair_store = a.d_vec16 && a.zf_h * a.zf_w == 1 && (a.Nout % 8 == 0 || a.pad_zero);  // uniform
    if (pair_store) {
        // Buffer stores: 32-bit offsets, and what must not be written passes an offset out of range (no branches).  They stay
        // in the caches, where the next layer reads them: with the non-temporal hint a call by itself is 5 % faster, the train
        // step of ResNet-50 1 % slower, pruned 15 % (lines written in two parts).
        const __amdgpu_buffer_rsrc_t d_srd = __builtin_amdgcn_make_buffer_rsrc(a.D, 0, kBufRecords, kBufFlags);
        const bool odd = (l32 & 1) != 0;
        const int ch0 = n0 + wn * WTN + (odd ? 16 : 0) + 8 * (lane >> 5);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const uint32_t m = (uint32_t)(m0 + wm * WTM + tm * 32 + (l32 & ~1));  // this lane stores to pixels m and m + 1
            uint32_t at0 = m * a.dst.point + a.dst.origin, at1 = at0 + a.dst.point;
            if (!a.d_linear) {  // uniform
                const uint32_t row0 = fdiv(m, a.gW), row1 = fdiv(m + 1, a.gW);
                at0 += row0 * a.dst.row + fdiv(row0, a.gH) * a.dst.image;
                at1 += row1 * a.dst.row + fdiv(row1, a.gH) * a.dst.image;
            }
            const bool ok0 = m < (uint32_t)a.M, ok1 = m + 1 < (uint32_t)a.M;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                if (n0 + wn * WTN + tn * 32 >= a.Nout) continue;  // wave-uniform
                const f32x16& c = acc[tn][tm];
                uint32_t v[2][4];  // this lane's chunk of each register pair: channels 16 gp + 8 (lane / 32) + {0..7} of the block
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) {
                    const uint32_t p0 = cvt_pk_bf16(c[8 * gp + 0], c[8 * gp + 1]), q0 = cvt_pk_bf16(c[8 * gp + 2], c[8 * gp + 3]);
                    const uint32_t p1 = cvt_pk_bf16(c[8 * gp + 4], c[8 * gp + 5]), q1 = cvt_pk_bf16(c[8 * gp + 6], c[8 * gp + 7]);
                    const auto ps = __builtin_amdgcn_permlane32_swap(p0, p1, false, false);
                    const auto qs = __builtin_amdgcn_permlane32_swap(q0, q1, false, false);
                    v[gp][0] = ps[0]; v[gp][1] = qs[0]; v[gp][2] = ps[1]; v[gp][3] = qs[1];
                }
                u32x4 o0, o1;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t got = swap_lane_pair(odd ? v[0][e] : v[1][e]);
                    o0[e] = odd ? got : v[0][e];
                    o1[e] = odd ? v[1][e] : got;
                }
                const int ch = ch0 + tn * 32;
                if (a.Nout % 8 != 0 && ch + 7 >= a.Nout) {  // last chunk of a zero-padded tensor: zeros in its padding
                    const Mask8 k = make_mask8(a.Nout - ch);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o0[e] &= k.m[e], o1[e] &= k.m[e];
                }
                const uint32_t at = (uint32_t)ch * 2u;
                __builtin_amdgcn_raw_buffer_store_b128(o0, d_srd, ok0 && ch < a.Nout ? at0 + at : kBufOut, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(o1, d_srd, ok1 && ch < a.Nout ? at1 + at : kBufOut, 0, 0);
            }
        }
    } else {
        const int hi = lane >> 5;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int m = m0 + wm * WTM + tm * 32 + l32;
            int64_t dpix;
            int cell_h = 1, cell_w = 1;  // pixels of this lane's cell inside the destination image
            if (a.d_linear) {
                dpix = (int64_t)m * a.dpitch;
            } else {
                const uint32_t mm = (uint32_t)min(m, a.M - 1);
                const uint32_t row = fdiv(mm, a.gW), gj = mm - row * a.gW.d;
                const uint32_t n = fdiv(row, a.gH), gi = row - n * a.gH.d;
                const int dh = (int)gi * a.d_hmul + a.d_hadd, dw = (int)gj * a.d_wmul + a.d_wadd;
                dpix = (((int64_t)n * a.DH + dh) * a.DW + dw) * a.dpitch;
                cell_h = min(a.zf_h, a.DH - dh);
                cell_w = min(a.zf_w, a.DW - dw);
            }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const int chb = n0 + wn * WTN + tn * 32;
                if (chb >= a.Nout) continue;  // wave-uniform
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) {  // register pairs (g = 2gp, 2gp + 1)
                    const f32x16& c = acc[tn][tm];
                    const uint32_t p0 = cvt_pk_bf16(c[8 * gp + 0], c[8 * gp + 1]), q0 = cvt_pk_bf16(c[8 * gp + 2], c[8 * gp + 3]);
                    const uint32_t p1 = cvt_pk_bf16(c[8 * gp + 4], c[8 * gp + 5]), q1 = cvt_pk_bf16(c[8 * gp + 6], c[8 * gp + 7]);
                    const auto ps = __builtin_amdgcn_permlane32_swap(p0, p1, false, false);
                    const auto qs = __builtin_amdgcn_permlane32_swap(q0, q1, false, false);
                    const int ch = chb + 16 * gp + 8 * hi;
                    if (m < a.M && ch < a.Nout) {
                        uint16_t* dst = a.D + dpix + ch;
                        if (a.zf_h * a.zf_w > 1) {  // uniform: clear the other pixels of the cell (vector stores only)
                            for (int zh = 0; zh < cell_h; ++zh)
                                for (int zw = zh == 0 ? 1 : 0; zw < cell_w; ++zw)
                                    *reinterpret_cast<uint4*>(dst + ((int64_t)zh * a.DW + zw) * a.dpitch) = make_uint4(0u, 0u, 0u, 0u);
                        }
                        if (a.d_vec16 && ch + 7 < a.Nout) {
                            *reinterpret_cast<uint4*>(dst) = make_uint4(ps[0], qs[0], ps[1], qs[1]);
                        } else if (a.d_vec16 && a.pad_zero && ch + 8 <= a.dpitch) {
                            // zero-padded tensors: the last chunk goes out as one vector too, zeros in its padding
                            *reinterpret_cast<uint4*>(dst) =
                                mask8(make_uint4(ps[0], qs[0], ps[1], qs[1]), true, make_mask8(a.Nout - ch));
                        } else {
                            const uint32_t w[4] = {ps[0], qs[0], ps[1], qs[1]};
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                if (ch + e < a.Nout) dst[e] = (uint16_t)(w[e >> 1] >> ((e & 1) * 16));
                        }
                    }
                }
            }
        }
    }
    if constexpr (STATS) {
        // Every lane holds 16 channel values per 32x32 block (channels 8g + 4*(lane/32) + i, v = 4g + i) of one
        // pixel.  A halving butterfly over the 32 pixel lanes of each half-wave leaves lane l with the total of the
        // one value v(l) = bits (16, 8, 4, 2) of l: 16 exchanges per block and statistic instead of 80.
        float* red = reinterpret_cast<float*>(smem_b);  // [2][WGM][BN]; the stage buffers are dead after the barrier
        __syncthreads();
        const int hi = lane >> 5;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            float sv[16], qv[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) sv[v] = 0.f, qv[v] = 0.f;
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const bool valid = m0 + wm * WTM + tm * 32 + l32 < a.M;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    // the value as stored: rounded to bf16
                    const float r = __uint_as_float(cvt_pk_bf16(acc[tn][tm][v], 0.f) << 16);
                    const float rv = valid ? r : 0.f;
                    sv[v] += rv;
                    qv[v] += rv * rv;
                }
            }
            static_for<0, 4>([&](auto step_c) {  // halves 8, 4, 2, 1 exchanged across lane bits 16, 8, 4, 2
                constexpr int HALF = 8 >> decltype(step_c)::value, BIT = 16 >> decltype(step_c)::value;
                const bool up = (l32 & BIT) != 0;
                static_for<0, HALF>([&](auto i_c) {
                    constexpr int I = decltype(i_c)::value;
                    const float ss = up ? sv[I] : sv[I + HALF], sq = up ? qv[I] : qv[I + HALF];
                    const float ks = up ? sv[I + HALF] : sv[I], kq = up ? qv[I + HALF] : qv[I];
                    sv[I] = ks + __shfl_xor(ss, BIT, 64);
                    qv[I] = kq + __shfl_xor(sq, BIT, 64);
                });
            });
            sv[0] += __shfl_xor(sv[0], 1, 64);
            qv[0] += __shfl_xor(qv[0], 1, 64);
            if ((l32 & 1) == 0) {
                const int v = ((l32 >> 4) & 1) * 8 + ((l32 >> 3) & 1) * 4 + ((l32 >> 2) & 1) * 2 + ((l32 >> 1) & 1);
                const int chl = wn * WTN + tn * 32 + 8 * (v >> 2) + 4 * hi + (v & 3);
                red[(0 * WGM + wm) * BN + chl] = sv[0];
                red[(1 * WGM + wm) * BN + chl] = qv[0];
            }
        }
        __syncthreads();
        for (int t = tid; t < 2 * BN; t += 64 * NW) {
            const int q = t / BN, chl = t - q * BN;
            if (n0 + chl >= a.Nout) continue;
            float tot = 0.f;
#pragma unroll
            for (int w = 0; w < WGM; ++w) tot += red[(q * WGM + w) * BN + chl];  // fixed order
            a.stats[((size_t)q * a.tiles_m + tile_m) * a.Nout + n0 + chl] = tot;
        }
    }
#endif
}

// What the host has decided for one problem of the direct kernel: which instantiation, and its launch shape.
typedef void (*igemm_dl_kern_t)(const IgemmArgsN);
struct IgemmDlPlan {
    // [0] the instantiation for this problem, [1] the same with the tap validity tests, [2] with the folded mode as well: what
    // a group of problems falls back to when only some of them could do without
    igemm_dl_kern_t kern[3];
    LdsOptIn* opt_in[3];
    size_t lds, lds_used;
    int threads;
};

// Problems that chose the same instantiation go out as ONE launch (blockIdx.y = problem): the tail of one overlaps the
// head of the next, and a group of short launches pays the fixed cost of a launch once.
inline hipError_t launch_igemm_dl_planned(const IgemmArgs* as, const IgemmDlPlan* ps, int n, hipStream_t st) {
    bool done[kIgemmMaxProblems] = {false, false, false, false};
    if (n > kIgemmMaxProblems) return hipErrorInvalidValue;
    // one launch of a more general instantiation rather than two of their own
    int level = 0;
    for (int l = 2; l >= 0; --l) {
        bool same = true;
        for (int i = 1; i < n; ++i) same = same && ps[i].kern[l] == ps[0].kern[l];
        if (same) level = l;
    }
    for (int i = 0; i < n; ++i) {
        if (done[i]) continue;
        IgemmArgsN m{};
        int cnt = 0, gx = 0;
        size_t lds_used = 0;
        for (int j = i; j < n; ++j) {
            if (done[j] || ps[j].kern[level] != ps[i].kern[level]) continue;
            done[j] = true;
            // longest workgroups first: the launch ends on short ones
            int at = cnt++;
            for (; at > 0 && m.a[at - 1].nk < as[j].nk; --at) m.a[at] = m.a[at - 1];
            m.a[at] = as[j];
            gx = as[j].grid_x > gx ? as[j].grid_x : gx;
            lds_used = ps[j].lds_used > lds_used ? ps[j].lds_used : lds_used;
        }
        const igemm_dl_kern_t kern = ps[i].kern[level];
        if (hipError_t e = ps[i].opt_in[level]->ensure(reinterpret_cast<const void*>(kern), ps[i].lds); e != hipSuccess) return e;
        // (several problems: a width that is a multiple of the 8 XCDs keeps every problem's tile -> XCD assignment)
        const unsigned gxr = cnt > 1 ? (unsigned)((gx + 7) / 8 * 8) : (unsigned)gx;
        hipLaunchKernelGGL(kern, dim3(gxr, (unsigned)cnt), dim3((unsigned)ps[i].threads), lds_used, st, m);
    }
    return hipSuccess;
}

// Offsets, tap intervals and tile division of the direct kernels, from the problem's geometry; `fast` = tiles along the axis
// that consecutive tiles run along.
inline void make_igemm_offsets(IgemmArgs& a, int fast) {
    a.t_div = make_fastdiv(fast);
    auto offsets = [&](int64_t point, int64_t row, int64_t image, int64_t origin) {  // of one step in j, i, n; in elements
        return RowOffsets{(uint32_t)(point * 2), (uint32_t)((row - a.gW.d * point) * 2), (uint32_t)((image - a.gH.d * row) * 2),
                          (uint32_t)(origin * 2)};
    };
    const int64_t ap = a.apitch, dp = a.dpitch;
    a.src = offsets(a.w_mul * ap, a.h_mul * a.srcW * ap, (int64_t)a.srcH * a.srcW * ap,
                    ((int64_t)a.h_add * a.srcW + a.w_add) * ap + a.a_guard);
    a.dst = offsets(a.d_wmul * dp, (int64_t)a.d_hmul * a.DW * dp, (int64_t)a.DH * a.DW * dp, ((int64_t)a.d_hadd * a.DW + a.d_wadd) * dp);
    // tap t reads source row h0 + t * step (step = +-1): inside for t in [-h0, -h0 + srcH) or [h0 - srcH + 1, h0 + 1)
    const bool hup = a.tr_step > 0, wup = a.ts_step > 0;
    a.ch_mul = hup ? -a.h_mul : a.h_mul;
    a.ch_add = hup ? -a.h_add : a.h_add - a.srcH + 1;
    a.cw_mul = wup ? -a.w_mul : a.w_mul;
    a.cw_add = wup ? -a.w_add : a.w_add - a.srcW + 1;
    a.tap_rep = 0;
    for (int r = 0; r < a.TR && r * a.TSm < 64; ++r) a.tap_rep |= 1ull << (r * a.TSm);
}

// Buffer addressing of the gathered operand (see k_igemm_dl): shifts that make both address parts non-negative; false if a
// tensor does not fit the 32-bit byte offsets.
inline bool igemm_buffer_args(IgemmArgs& a) {
    a.a_guard = ((a.h_add < 0 ? -a.h_add : 0) * a.srcW + (a.w_add < 0 ? -a.w_add : 0)) * a.apitch;
    const int last_r = (a.TR - 1) * a.tr_step, last_s = (a.TS - 1) * a.ts_step;
    a.a_smin = ((last_r < 0 ? last_r : 0) * a.srcW + (last_s < 0 ? last_s : 0)) * a.apitch;
    const int64_t img = (int64_t)ceil_div(a.M, (int64_t)a.gH.d * a.gW.d);  // images of the source tensor
    return (img * a.srcH * a.srcW * a.apitch + a.a_guard) * 2 < 0xffffff00ll && (int64_t)a.Nout * a.b_taps * a.bpitch * 2 < 0xffffff00ll;
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool DEEP = false>
inline hipError_t plan_igemm_dl_cfg(IgemmArgs& a, IgemmDlPlan& plan) {
    constexpr int NT = 64 * WGM * WGN;
    constexpr size_t lds = (size_t)STAGES * (BM + BN) * 128;
    static_assert(lds <= 160 * 1024, "LDS capacity");
    // last channel block of a tap is short and/or some chunk has a masked tail
    const bool ragged = (a.Cred % 64) != 0 || (a.fold && a.Creal % 8 != 0);
    a.nk = a.TR * a.TS * (int)ceil_div(a.CredP, 64);  // steps are (tap, block of 64 channels)
    a.tiles_n = (int)ceil_div(a.Nout, BN);
    set_tail_tables(a);
    // variant: 0 = whole 64-channel blocks, 1 = partial blocks but no undefined elements (channel count a multiple
    // of 8, or the caller vouches for zero padding), 2 = partial blocks with tails to clear
    int variant = !ragged ? 0 : (a.tail_kv == 0 || a.pad_zero ? 1 : 2);
    if (a.stats) {  // statistics epilogue: variants 3, 4 = variants 0, 1 with it (the caller has ruled out tails)
        if (variant == 2) return hipErrorInvalidValue;
        variant += 3;
    }
    a.tiles_m = (int)ceil_div(a.M, BM);
    if (DEEP && (variant > 1 || a.fold || a.nk < STAGES)) return hipErrorInvalidValue;
    if (!igemm_buffer_args(a)) return hipErrorInvalidValue;
    // every tap of every row inside the source image?  coordinates are monotone in the grid index and in the tap
    auto inside = [](int lo, int hi, int n) { return lo >= 0 && hi >= 0 && lo < n && hi < n; };
    const int h_first = a.h_add, h_last = ((int)a.gH.d - 1) * a.h_mul + a.h_add;
    const int w_first = a.w_add, w_last = ((int)a.gW.d - 1) * a.w_mul + a.w_add;
    const int rr = (a.TR - 1) * a.tr_step, ss = (a.TSm - 1) * a.ts_step;
    a.a_all_valid = inside(h_first, h_last, a.srcH) && inside(h_first + rr, h_last + rr, a.srcH) &&
                    inside(w_first, w_last, a.srcW) && inside(w_first + ss, w_last + ss, a.srcW);
    const bool av = a.a_all_valid && variant != 2;
    // (the deep form: no tails, no statistics, no folded mode)
    constexpr bool D = DEEP, T = !DEEP;
    static const igemm_dl_kern_t kerns[3][5] = {{k_igemm_dl<BM, BN, WGM, WGN, STAGES, false, false, false, false, false, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, false, false, false, false, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, T, false, false, false, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, false, false, T, false, false, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, false, T, false, false, D>},
                                                {k_igemm_dl<BM, BN, WGM, WGN, STAGES, false, false, false, true, false, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, false, false, true, false, D>,
                                                 nullptr,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, false, false, T, true, false, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, false, T, true, false, D>},
                                                {k_igemm_dl<BM, BN, WGM, WGN, STAGES, false, false, false, false, T, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, false, false, false, T, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, T, false, false, T, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, false, false, T, false, T, D>,
                                                 k_igemm_dl<BM, BN, WGM, WGN, STAGES, true, false, T, false, T, D>}};
    static LdsOptIn opt_in[3][5];
    const int tests = a.fold ? 2 : 0, rows[3] = {av ? 1 : tests, tests, 2};
    for (int l = 0; l < 3; ++l) {
        plan.kern[l] = kerns[rows[l]][variant];
        plan.opt_in[l] = &opt_in[rows[l]][variant];
    }
    plan.lds = lds;
    plan.threads = NT;
    const int64_t tiles = ceil_div(a.M, BM) * a.tiles_n;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    a.grid_x = (int)tiles;
    make_igemm_offsets(a, a.tiles_n);
    // A reduction of fewer steps than the pipeline has stages touches only the first nk stage buffers (and the
    // statistics epilogue a few KB of the first): the launch asks for no more LDS than that, which leaves room on the
    // CU for workgroups of kernels running beside it (train step at pruned widths -0.6 %, full -0.2 %).
    plan.lds_used = (size_t)(a.nk < STAGES ? (a.nk < 1 ? 1 : a.nk) : STAGES) * (BM + BN) * 128;
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------- //
// forward / input-gradient implicit GEMM with few output tiles
// ------------------------------------------------------------------------------------------- //
// A problem with few tiles (a small batch, a late layer) leaves most of the chip idle in k_igemm_dl, and each of its
// workgroups is a serial chain of reduction steps that hides nothing.  Here the eight waves of a workgroup share one SMALL
// tile (32 x 32 or 64 x 64 outputs) and divide the REDUCTION between them: a stage is NB steps of 64 channels at once,
// every wave multiplies its own part of it, and the partial tiles are added through LDS in a fixed order at the end.  Four
// to sixteen times the workgroups, a quarter or half of the barriers.  Operand traffic per flop is two to four times that
// of the large tiles, which is why they keep the problems that fill the chip.
// Same arguments, addressing and LDS layout as k_igemm_dl (one 64-channel step = BM + BN rows of 128 bytes, chunks XOR-ed
// with the row), every geometry in one instantiation: a bit per tap (at most 31 of them) is tested per load.  No TAIL
// (undefined channel padding), no statistics.
// Bound by a wave's own instructions, one after the other, between two barriers: wait, fragment reads, loads, two MFMAs or one.
// The fragments are read ahead of the issue of a later stage's loads, and what only a tap's end changes stands behind a branch
// (see issue): 7 x 7 333 -> 300, 3 x 3, batch 10: 11.2 -> 8.0 us, 14 x 14 650 -> 170, 1 x 1: 6.5 -> 5.8.  64 x 64 tiles move half
// as much per flop as 32 x 32.  Both take 64 KB in four stages, two workgroups on the CU: 64 x 64 from memory in three stages 14 x
// 14 256 -> 256 11.1 us, in four 10.1, in five 10.3, with two steps a stage 10.2 and 13.6; 32 x 32 in fours of steps in
// three stages (96 KB, one on the CU) 14 x 14 171 -> 165 10.3 us, in pairs in four 8.2.
template <int BM, int BN, int NB, int STAGES>
__global__ __launch_bounds__(512, 1) void k_igemm_small(const IgemmArgsN problems) {
#if defined(__HIP_DEVICE_COMPILE__)
    const IgemmArgs a = problems.a[blockIdx.y];
    if (a.edge_prio) __builtin_amdgcn_s_setprio(2);
    constexpr int NW = 8, WT = (BM / 32) * (BN / 32), KS = NW / WT;  // waves over the tile, parts of the reduction
    constexpr int LPW = (BM + BN) / 64;                             // loads per wave and step
    constexpr int SUB = (BM + BN) * 128, STAGE = NB * SUB;
    constexpr int PER = NB * 4 / KS;                                // 16-channel sub-steps per wave and stage
    static_assert(WT * KS == NW && (BM / 8) % 2 == 0 && PER >= 1 && (PER <= 4 ? 4 % PER == 0 : PER % 4 == 0), "tile config");
    static_assert(STAGES >= 2 && (STAGES - 1) * LPW * NB < 64, "stages");
    constexpr int RP = BN + 4;  // row pitch of the partial tiles, floats
    static_assert(KS * BM * RP * 4 <= STAGES * STAGE, "partial tiles");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_b[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = xcd_remap(blockIdx.x, a.grid_x);
    const int slow = (int)fdiv((uint32_t)tile, a.t_div), fast = tile - slow * (int)a.t_div.d;
    const int m0 = (a.m_fast ? fast : slow) * BM, n0 = (a.m_fast ? slow : fast) * BN;

    // Loads as in k_igemm_dl: per-lane constants in voffset, running scalar offsets in soffset, one bit per tap and
    // lane.  A wave's load j is of one operand: the roles are scalar selects, and both operands take the same instructions.
    const int lrow = lane >> 3;
    constexpr uint32_t kBufRecords = 0xffffff00u, kBufOut = 0xffffffffu, kBufFlags = 0x00020000u;
    const int nblk = (a.CredP + 63) / 64, back = (nblk - 1) * 128;
    uint32_t voff[LPW], now[LPW], past[LPW], soff[LPW];  // now: voff, or kBufOut if the tap reads zeros; past: all ones if ...
    int col_d[LPW], row_d[LPW], skip[LPW];               // ... the last block of a tap does; skip: a bit per tap that does
    int kvoff[LPW];
    __amdgpu_buffer_rsrc_t srd[LPW];
    auto flag = [](int bits) { return (uint32_t)(bits << 31 >> 31); };  // bit 0, in all bits
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
        const int g = wave + NW * j;  // 8-row group of the step: the first BM / 8 are pixels
        kvoff[j] = ((lane & 7) ^ (((g & 1) << 2) | (lane >> 4))) * 8;
        if (g < BM / 8) {  // uniform
            const uint32_t m = (uint32_t)min(m0 + g * 8 + lrow, a.M - 1);
            const uint32_t row = fdiv(m, a.gW), n = fdiv(row, a.gH);
            voff[j] = m * a.src.point + row * a.src.row + n * a.src.image + a.src.origin + (uint32_t)kvoff[j] * 2u;
            skip[j] = tap_skip(a, (int)(row - n * a.gH.d), (int)(m - row * a.gW.d)).lo;
        } else {
            const int nrow = min(n0 + (g - BM / 8) * 8 + lrow, a.Nout - 1);
            voff[j] = ((uint32_t)nrow * ((uint32_t)a.b_taps * a.bpitch) + (uint32_t)kvoff[j]) * 2u;
            skip[j] = (int)(~0u << (a.TR * a.TSm));
        }
        now[j] = voff[j] | flag(skip[j]);
        past[j] = (nblk - 1) * 64 + kvoff[j] < a.Cred ? 0u : kBufOut;
        const bool px = g < BM / 8;
        const uint16_t* base = px ? a.A + ((int64_t)a.a_smin - a.a_guard) : a.B;  // uniform
        srd[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, kBufRecords, kBufFlags);
        const int ts_d = px ? a.ts_step * a.apitch * 2 : a.b_ts_stride * a.bpitch * 2;
        col_d[j] = ts_d - back;
        row_d[j] = (px ? a.tr_step * a.srcW * a.apitch * 2 : a.b_tr_stride * a.bpitch * 2) - (a.TS - 1) * ts_d - back;
        soff[j] = (uint32_t)(px ? -a.a_smin * 2 : a.b_tap0 * a.bpitch * 2);
    }
    // Sends out one stage.  What only a tap's end changes stands behind a branch, at the end of a step: a wave's own instructions,
    // one after the other, are what a step takes (70 of them 0.24 us), and with the branch there are 30.
    int blk = nblk, col = a.TS, f_cb = 0;
    auto issue = [&](int at) {  // at: byte offset of the stage
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            uint8_t* sbase = smem_b + at + b * SUB;
            const uint32_t last = blk == 1 ? ~0u : 0u;
#pragma unroll
            for (int j = 0; j < LPW; ++j) {
                uint32_t v = now[j];
                if (a.fold) v = voff[j] | flag(skip[j] >> ((int)fdiv((uint32_t)(f_cb + kvoff[j]), a.Cfold) & 31));  // uniform: the tap depends on the lane's chunk
                __builtin_amdgcn_raw_ptr_buffer_load_lds(srd[j], (lds_void_ptr)(sbase + (wave + NW * j) * 1024), 16, v | (past[j] & last), soff[j], 0, 0);
                soff[j] += 128u;
            }
            f_cb += 64;
            if (--blk == 0) {  // uniform (past the last step every tap reads zeros: skip is sign-extended)
                const bool last_col = --col == 0;
#pragma unroll
                for (int j = 0; j < LPW; ++j) {
                    soff[j] += (uint32_t)((last_col ? row_d[j] : col_d[j]) - 128);
                    skip[j] >>= a.fold ? a.TSm : 1;  // folded: a filter row
                    now[j] = voff[j] | flag(skip[j]);
                }
                blk = nblk;
                col = last_col ? a.TS : col;
                f_cb = 0;
            }
        }
    };
    const int kg = wave / WT, wt = wave - kg * WT;  // part of the reduction, block of the tile
    const int wm = wt % (BM / 32), wn = wt / (BM / 32);
    const int l32 = lane & 31, swz = (l32 >> 1) & 7, kc0 = lane >> 5;
    const int ss0 = (kg * PER) & 3;
    const int a_row = ((kg * PER) >> 2) * SUB + (wm * 32 + l32) * 128, b_row = ((kg * PER) >> 2) * SUB + (BM + wn * 32 + l32) * 128;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;

    if (blockIdx.x >= (unsigned)a.grid_x) return;  // the whole workgroup
    const int nst = (a.nk + NB - 1) / NB;
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue(s * STAGE);
    for (int st0 = 0; st0 < nst; st0 += STAGES) {
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            if (st0 + s < nst) {
                wait_vmcnt<(STAGES - 2) * LPW * NB>();
                barrier_nofence();
                // fragments first: the loads of a later stage are sent out while these are on their way
                const uint8_t* base = smem_b + s * STAGE;
                bf16x8 fa[PER], fb[PER];
#pragma unroll
                for (int q = 0; q < PER; ++q) {
                    const int off = (q >> 2) * SUB + ((((ss0 + (q & 3)) * 2 + kc0) ^ swz) << 4);
                    fb[q] = *reinterpret_cast<const bf16x8*>(base + b_row + off);
                    fa[q] = *reinterpret_cast<const bf16x8*>(base + a_row + off);
                }
                issue((s + STAGES - 1) % STAGES * STAGE);  // (past the end: zeros into a stage nobody multiplies)
#pragma unroll
                for (int q = 0; q < PER; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[q], fa[q], acc, 0, 0, 0);
            }
        }
    }
    wait_vmcnt<0>();
    __syncthreads();
    // partial tiles: lane holds pixel l32, channels 8 g + 4 (lane / 32) + {0..3} of its 32 x 32 block
    float* red = reinterpret_cast<float*>(smem_b);
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(red + (kg * BM + wm * 32 + l32) * RP + wn * 32 + 8 * g + 4 * kc0) =
            make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
    __syncthreads();
    // every thread adds and stores E consecutive channels of one pixel (32 x 32: all 512 of them, not 128 with eight each)
    constexpr int E = BM * BN / 512, TPP = BN / E;
    static_assert(E == 2 || E == 8, "elements per thread");
    const int px = tid / TPP, chl = (tid % TPP) * E, ch = n0 + chl, m = m0 + px;
    const float* src = red + px * RP + chl;
    float v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src[e];
#pragma unroll
    for (int g = 1; g < KS; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] += src[g * BM * RP + e];
    uint32_t at = (uint32_t)m * a.dst.point + a.dst.origin + (uint32_t)ch * 2u;
    int cell_h = 1, cell_w = 1;
    if (!a.d_linear) {  // uniform
        const uint32_t row = fdiv((uint32_t)m, a.gW), n = fdiv(row, a.gH);
        at += row * a.dst.row + n * a.dst.image;
        cell_h = min(a.zf_h, a.DH - ((int)(row - n * a.gH.d) * a.d_hmul + a.d_hadd));
        cell_w = min(a.zf_w, a.DW - ((int)(m - row * a.gW.d) * a.d_wmul + a.d_wadd));
    }
    typedef uint32_t vec_t __attribute__((ext_vector_type(E / 2)));
    vec_t o;
    uint16_t* dst = reinterpret_cast<uint16_t*>(reinterpret_cast<uint8_t*>(a.D) + at);
    if (m >= a.M || ch >= (a.pad_zero ? (int)((a.Nout + 7) & ~7) : a.Nout)) return;
    if (a.zf_h * a.zf_w > 1) {  // uniform: clear the other pixels of the cell (vector stores only)
#pragma unroll
        for (int e = 0; e < E / 2; ++e) o[e] = 0u;
        for (int zh = 0; zh < cell_h; ++zh)
            for (int zw = zh == 0 ? 1 : 0; zw < cell_w; ++zw)
                *reinterpret_cast<vec_t*>(dst + ((int64_t)zh * a.DW + zw) * a.dpitch) = o;
    }
#pragma unroll
    for (int e = 0; e < E / 2; ++e) o[e] = cvt_pk_bf16(v[2 * e], v[2 * e + 1]);
    // whole chunks of eight channels, of a zero-padded tensor also the last one (zeros in its padding), as vectors
    if (a.d_vec16 && ((ch | 7) < a.Nout || (a.pad_zero && (ch | 7) < a.dpitch))) {
        if (ch + E > a.Nout) {
#pragma unroll
            for (int e = 0; e < E / 2; ++e) {
                const int k = a.Nout - ch - 2 * e;
                o[e] &= k >= 2 ? 0xffffffffu : k == 1 ? 0xffffu : 0u;
            }
        }
        *reinterpret_cast<vec_t*>(dst) = o;
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (ch + e < a.Nout) dst[e] = (uint16_t)(o[e >> 1] >> ((e & 1) * 16));
    }
#endif
}

template <int BM, int BN, int NB, int STAGES>
inline hipError_t plan_igemm_small_cfg(IgemmArgs& a, IgemmDlPlan& plan) {
    constexpr size_t lds = (size_t)STAGES * NB * (BM + BN) * 128;
    static_assert(lds <= 160 * 1024, "LDS capacity");
    a.nk = a.TR * a.TS * (int)ceil_div(a.CredP, 64);
    a.tiles_n = (int)ceil_div(a.Nout, BN);
    a.tiles_m = (int)ceil_div(a.M, BM);
    if (!igemm_buffer_args(a)) return hipErrorInvalidValue;
    // neighbouring tiles, which share an XCD and its L2, should share the larger operand
    a.m_fast = (int64_t)a.Nout * a.b_taps * a.bpitch > (int64_t)a.M * a.CredP;
    static LdsOptIn opt_in;
    for (int l = 0; l < 3; ++l) {
        plan.kern[l] = k_igemm_small<BM, BN, NB, STAGES>;
        plan.opt_in[l] = &opt_in;
    }
    plan.lds = plan.lds_used = lds;
    plan.threads = 512;
    const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    a.grid_x = (int)tiles;
    make_igemm_offsets(a, a.m_fast ? a.tiles_m : a.tiles_n);
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------- //
// forward convolution of a network's first layer: image-like input, at most 4 channels at a pitch of 8
// ------------------------------------------------------------------------------------------- //
// The implicit-GEMM kernel treats such a layer as a GEMM over folded filter rows of S * 8 elements: 5 of every 8
// multiplied elements are padding, and every output pixel pulls R runs of S pixels from L2 into LDS again.  Here a
// workgroup walks over a run of tiles of 4 x 64 output pixels (x 64 output channels).  It keeps ALL its weights in
// registers for the whole run (a filter row is 8 taps x 4 channels = two 16-element MFMA steps; taps past S and
// channels past C are zero).  Per tile it loads the input patch under the tile ONCE, 8 bytes (4 channels) per pixel,
// into LDS in image order: the two taps a lane multiplies in one step are neighbouring pixels, 16 contiguous bytes, and
// consecutive output pixels read consecutive (stride 1) or every other (stride 2) such pair.  The patch of the next
// tile is fetched into registers before the current tile is multiplied and written to the other of two LDS buffers
// after it, so that its memory latency hides behind the MFMAs.  R * 2 MFMAs per 32 x 32 block: against the folded
// form half the matrix work and an eighth of the operand traffic.  Both operands' padding channels must be zero (the
// caller's PT_CONV_PAD_ZERO), the output takes 16-byte stores.
struct StemArgs {
    const uint16_t* X;   // [N][H][W][8]
    const uint16_t* Wt;  // [K][R][S][8]
    uint16_t* Y;         // [N][P][Q][ypitch]
    int N, H, W, P, Q, K, R, S, pad_h, pad_w, ypitch;
    int tiles_q, tiles_p;  // tiles per image along Q and P
    int tiles, run;        // N * tiles_p * tiles_q, and how many consecutive tiles one workgroup takes
};
constexpr int kStemTH = 4, kStemTW = 64, kStemMaxR = 8;
constexpr int kStemSlots = 512;  // 256 CUs x 2 resident workgroups

// RT: rows of the filter the multiply loop runs over (R itself, or 8 for any R <= 8: rows past R multiply zeros);
// NJ: 16-element steps per filter row (1 for S <= 4, else 2).
template <int STRIDE, int RT, int NJ>
__global__ __launch_bounds__(512, 4) void k_stem_fwd(const StemArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int PH = (kStemTH - 1) * STRIDE + RT;              // patch rows
    constexpr int PW = (kStemTW - 1) * STRIDE + 4 * NJ;          // patch columns: 4 taps per step
    constexpr int PWR = (PW + 1) & ~1;                           // row pitch in pixels: rows start on 16 bytes
    constexpr int PSZ = PH * PWR;
    __shared__ __attribute__((aligned(16))) uint2 patch[2][PSZ]; // [buffer][row][column], 4 channels each
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_n = (a.K + 63) / 64;
    const int nt = blockIdx.x % tiles_n, chunk = blockIdx.x / tiles_n;
    const int n0 = nt * 64;
    const int first = chunk * a.run, last = first + a.run < a.tiles ? first + a.run : a.tiles;
    if (first >= last) return;  // whole workgroup
    const int ph_used = (kStemTH - 1) * STRIDE + a.R;            // rows of the patch this filter reaches (<= PH)

    // ---- weights -> registers: fragment (r, j) of this lane = taps 4j + 2h, 4j + 2h + 1 of filter row r, 4 channels each
    const int wm = wave & 3, wn = wave >> 2;      // tile row of this wave, half of the 64 output channels
    const int l32 = lane & 31, h = lane >> 5;
    const int n = n0 + wn * 32 + l32;             // output channel of this lane's weight rows
    const bool n_ok = n < a.K;
    bf16x8 wf[RT][NJ];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            uint2 lo = make_uint2(0u, 0u), hi = make_uint2(0u, 0u);
            const int s0 = 4 * j + 2 * h;
            if (n_ok && r < a.R) {
                const uint16_t* wr = a.Wt + ((int64_t)(n * a.R + r) * a.S) * 8;
                if (s0 < a.S) lo = *reinterpret_cast<const uint2*>(wr + s0 * 8);
                if (s0 + 1 < a.S) hi = *reinterpret_cast<const uint2*>(wr + (s0 + 1) * 8);
            }
            wf[r][j] = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
        }

    // ---- this thread's pixels of a patch: LDS slots tid + 512 * it, the same in every tile --------------------------
    // (their rows and columns are worked out again at every use, from a copy of the thread index that the compiler
    // cannot see through: kept across the tile loop they cost registers, which spill)
    constexpr int NLD = (PSZ + 511) / 512;
    uint2 pv[NLD];
    // All loads of a patch are issued back to back, as buffer loads on a descriptor of the tile's image: a pixel
    // outside the image, or in a row the filter does not reach, passes an offset past the descriptor's range and reads
    // zeros (no branch, no cleared register, so nothing the loads would have to wait for).
    constexpr uint32_t kBufOut = 0xffffffffu, kBufFlags = 0x00020000u;
    const uint32_t img_bytes = (uint32_t)(a.H * a.W) * 16u;
    auto fetch = [&](int tq, int tp, int img) {
        const int ih0 = tp * kStemTH * STRIDE - a.pad_h, iw0 = tq * kStemTW * STRIDE - a.pad_w;
        const __amdgpu_buffer_rsrc_t x_srd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(a.X) + (int64_t)img * a.H * a.W * 8, 0, img_bytes, kBufFlags);
        int t0 = tid;
        asm volatile("" : "+v"(t0));
#pragma unroll
        for (int it = 0; it < NLD; ++it) {
            const int i = t0 + it * 512;
            const int prow = i / PWR, pcol = i - prow * PWR;
            const int ih = ih0 + prow, iw = iw0 + pcol;
            const bool ok = prow < ph_used && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;  // (rows >= PH: too)
            const auto got = __builtin_amdgcn_raw_buffer_load_b64(x_srd, ok ? (uint32_t)(ih * a.W + iw) * 16u : kBufOut, 0, 0);
            pv[it] = make_uint2(got[0], got[1]);
        }
    };
    auto park = [&](int buf) {
        int t0 = tid;
        asm volatile("" : "+v"(t0));
#pragma unroll
        for (int it = 0; it < NLD; ++it)
            if ((it + 1) * 512 <= PSZ || t0 + it * 512 < PSZ) patch[buf][t0 + it * 512] = pv[it];
    };
    // tiles are numbered (image, tile row, tile column), column fastest: the next one by counting up
    auto advance = [&](int& tq, int& tp, int& img) {
        if (++tq == a.tiles_q) {
            tq = 0;
            if (++tp == a.tiles_p) {
                tp = 0;
                ++img;
            }
        }
    };
    int ntq = first % a.tiles_q, ntp = (first / a.tiles_q) % a.tiles_p, nimg = first / (a.tiles_q * a.tiles_p);

    fetch(ntq, ntp, nimg);
    park(0);
    __syncthreads();
    const bool wave_n_live = n0 + wn * 32 < a.K;  // uniform
    // LDS element this lane's fragments start from: pixel l32 of the wave's tile row, tap 2h
    const int frag0 = wm * STRIDE * PWR + l32 * STRIDE + 2 * h;
    int buf = 0;
    for (int tile = first; tile < last; ++tile, buf ^= 1) {
        const bool more = tile + 1 < last;  // uniform
        const int tq = ntq, tp = ntp, img = nimg;
        advance(ntq, ntp, nimg);
        if (more) fetch(ntq, ntp, nimg);
        const int p = tp * kStemTH + wm, q0 = tq * kStemTW;
        const bool live = wave_n_live && p < a.P;  // uniform
        f32x16 acc[2];
        if (live) {
            // ---- multiply: this wave's 64 output pixels (tile row wm) x 32 output channels -------------------------
#pragma unroll
            for (int tm = 0; tm < 2; ++tm)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[tm][v] = 0.f;
            const uint2* pb = patch[buf] + frag0;
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int tm = 0; tm < 2; ++tm) {
                        // taps 4j + 2h, 4j + 2h + 1 of filter row r under output pixel tm * 32 + l32: two neighbouring pixels
                        const uint2* src = pb + r * PWR + tm * 32 * STRIDE + 4 * j;
                        uint4 x4;
                        if constexpr (STRIDE == 2) {
                            x4 = *reinterpret_cast<const uint4*>(src);  // an even column: 16-byte aligned
                        } else {
                            const uint2 lo = src[0], hi = src[1];
                            x4 = make_uint4(lo.x, lo.y, hi.x, hi.y);
                        }
                        acc[tm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[r][j], __builtin_bit_cast(bf16x8, x4), acc[tm], 0, 0, 0);
                    }
        }
        // The next patch goes to the other buffer (last read before the barrier that ended the previous tile) BEFORE this
        // tile's stores are issued: the wait for its loads then does not also wait for the stores behind them.
        if (more) park(buf ^ 1);
        if (live) {
            // ---- store: the lane-pair exchange of k_igemm_dl (64 contiguous bytes of 16 pixels per store instruction) ----
            // (a uniform base per tile and wave plus one 32-bit offset per lane; lane-derived values of this part are
            // worked out afresh per tile, not kept in registers across the multiply)
            const __amdgpu_buffer_rsrc_t y_srd = __builtin_amdgcn_make_buffer_rsrc(
                a.Y + ((int64_t)(img * a.P + p) * a.Q + q0) * a.ypitch + n0 + wn * 32, 0, 0xffffff00u, kBufFlags);
            int le = lane;
            asm volatile("" : "+v"(le));
            const int l32e = le & 31;
            const bool odd = (le & 1) != 0;
            const int chl = (odd ? 16 : 0) + 8 * (le >> 5);             // channel of this lane's chunk within the wave's 32
            const int ch = n0 + wn * 32 + chl;
#pragma unroll
            for (int tm = 0; tm < 2; ++tm) {
                const int q = q0 + tm * 32 + l32e;
                const uint32_t off0 = (uint32_t)((tm * 32 + (l32e & ~1)) * a.ypitch + chl) * 2u;  // pixel (q & ~1); (q | 1) is next
                const bool ok0 = (q & ~1) < a.Q, ok1 = (q | 1) < a.Q;
                const f32x16& c = acc[tm];
                uint32_t v[2][4];
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) {
                    const uint32_t x0 = cvt_pk_bf16(c[8 * gp + 0], c[8 * gp + 1]), y0 = cvt_pk_bf16(c[8 * gp + 2], c[8 * gp + 3]);
                    const uint32_t x1 = cvt_pk_bf16(c[8 * gp + 4], c[8 * gp + 5]), y1 = cvt_pk_bf16(c[8 * gp + 6], c[8 * gp + 7]);
                    const auto ps = __builtin_amdgcn_permlane32_swap(x0, x1, false, false);
                    const auto qs = __builtin_amdgcn_permlane32_swap(y0, y1, false, false);
                    v[gp][0] = ps[0]; v[gp][1] = qs[0]; v[gp][2] = ps[1]; v[gp][3] = qs[1];
                }
                uint32_t s0[4], s1[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t give = odd ? v[0][e] : v[1][e];
                    const uint32_t got = (uint32_t)__shfl_xor((int)give, 1, 64);
                    s0[e] = odd ? got : v[0][e];
                    s1[e] = odd ? v[1][e] : got;
                }
                uint4 o0 = make_uint4(s0[0], s0[1], s0[2], s0[3]), o1 = make_uint4(s1[0], s1[1], s1[2], s1[3]);
                if (ch < a.K && ch + 7 >= a.K) {  // last chunk: zeros in its padding
                    const Mask8 k = make_mask8(a.K - ch);
                    o0 = mask8(o0, true, k);
                    o1 = mask8(o1, true, k);
                }
                // (a pixel past the row's end, a chunk past the channel count: an offset out of range, the store is dropped)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o0), y_srd, ok0 && ch < a.K ? off0 : kBufOut, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o1), y_srd,
                                                       ok1 && ch < a.K ? off0 + (uint32_t)a.ypitch * 2u : kBufOut, 0, 0);
            }
        }
        __syncthreads();
    }
#endif
}

// One run of tiles per workgroup slot of the chip (2 workgroups per CU): the weights are fetched once per run.
inline hipError_t launch_stem_fwd(StemArgs& a, int stride, int slots, hipStream_t st) {
    a.tiles_q = (a.Q + kStemTW - 1) / kStemTW;
    a.tiles_p = (a.P + kStemTH - 1) / kStemTH;
    const int64_t tiles = (int64_t)a.N * a.tiles_p * a.tiles_q;
    if (tiles <= 0) return hipSuccess;
    if (tiles > 0x3fffffff) return hipErrorInvalidValue;
    a.tiles = (int)tiles;
    a.run = (int)((tiles + slots - 1) / slots);
    const int64_t grid = ((tiles + a.run - 1) / a.run) * ((a.K + 63) / 64);
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 g((unsigned)grid), b(512);
    const int nj = a.S <= 4 ? 1 : 2;
#define PT_STEM_CASE(ST, RT, NJ) hipLaunchKernelGGL((k_stem_fwd<ST, RT, NJ>), g, b, 0, st, a)
    if (stride == 1) {
        if (a.R == 3 && nj == 1) PT_STEM_CASE(1, 3, 1);
        else if (a.R == 7 && nj == 2) PT_STEM_CASE(1, 7, 2);
        else PT_STEM_CASE(1, 8, 2);
    } else {
        if (a.R == 3 && nj == 1) PT_STEM_CASE(2, 3, 1);
        else if (a.R == 7 && nj == 2) PT_STEM_CASE(2, 7, 2);
        else PT_STEM_CASE(2, 8, 2);
    }
#undef PT_STEM_CASE
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------- //
// weight gradient
// ------------------------------------------------------------------------------------------- //
struct WgradArgs {
    const uint16_t* X;   // x[N][H][W][xpitch]
    const uint16_t* DY;  // dy[pixels][ypitch]
    float* OUT;          // splits > 1: partial[split][K][Mtot]; else dw[K][RS][wpitch]
    int pixels;          // N*P*Q
    FastDiv Q, P;
    int H, W, xpitch, ypitch;
    int stride_h, stride_w, pad_h, pad_w;
    int S, RS, C, CP;    // CP = C rounded up to 8; Mtot = RS*CP
    int Mtot, K;
    int tiles_n;         // tiles along K
    int tiles_m;         // tiles along (tap, c)
    int tiles_per_tap;   // direct kernel: channel blocks per filter tap
    int KP;              // K rounded up to 8
    int fold;            // direct kernel: a tile row block spans the S taps of one filter row (dense small-C pixels)
    int iters_total, iters_per_split, splits;
    int dn, dp, dq;      // direct kernel: one reduction step of BKP pixels = dn images + dp output rows + dq output columns
    int cfg;             // direct kernel: tile configuration
    int xmode;           // direct kernel: 1 = stride 1 and output grid == input grid: x sits at (pixel + tap shift) * xpitch;
                         // 2 = in addition no tap ever leaves the image (1 x 1 filter without padding); 0 = any geometry
    // direct kernel writing dw itself (direct != 0): when lw is set, the gradient of the group-lasso penalty is added
    // to every element on the way out, dw += l_lambda * (lw * (1/l_on[k] + 1/l_in[c])) with a zero norm contributing 0
    const float* lw;    // fp32 master weights, layout and pitch of dw
    const float* l_on;  // [K], nullptr = output groups not regularised
    const float* l_in;  // [C], nullptr = input groups not regularised
    float l_lambda;
    int out_row_pitch;   // elements between consecutive k in the partial buffer (Mtot)
    int wpitch;
    int direct;          // 1: write dw layout directly (splits == 1)
    int o_vec;
    FastDiv ntile_div, tn_div, tap_div, S_div, CP_div;  // direct kernel: by tiles_m * tiles_n, tiles_n, tiles_per_tap, S, CP
    SmallDiv sQ, sP;     // register-staged kernel: Q, P
};

template <int BM, int BN, int BK, int WGM, int WGN, int MINB, bool VEC>
__global__ __launch_bounds__(64 * WGM * WGN, MINB) void k_wgrad(const WgradArgs a) {
    // LDS tiles are [pixel][channel] with a row pad of 32 elements (64 bytes): the four pixel rows a
    // 16-lane group touches in one transpose read then fall into different banks.
    constexpr int NT = 64 * WGM * WGN;
    constexpr int LDM = BM + 32, LDN = BN + 32;
    constexpr int XV = BM / 8, YV = BN / 8;  // 8-vectors per pixel row
    constexpr int XR = NT / XV, YR = NT / YV;  // pixel rows per pass
    constexpr int XP = BK / XR, YP = BK / YR;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    constexpr int STAGE_ELEMS = BK * (LDM + LDN);
    static_assert(XP >= 1 && YP >= 1 && TM >= 1 && TN >= 1 && BK % 16 == 0 && BK % XR == 0 && BK % YR == 0, "tile config");
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction
    // Workgroup ids are dealt round-robin to the 8 XCDs.  All tiles of one pixel split read the same x and dy
    // slabs, so each XCD gets a contiguous range of the split-major (split, tile) order: a split's tiles run
    // back to back on one XCD and the slabs are fetched into that L2 once.
    const int ntile = a.tiles_m * a.tiles_n;
    const int lin = xcd_remap(blockIdx.x, gridDim.x);
    const int split = lin / ntile;
    const int tile = lin - split * ntile;
    const int n0 = (tile % a.tiles_n) * BN;  // k origin
    const int m0 = (tile / a.tiles_n) * BM;  // (tap, c) origin
    const int it0 = split * a.iters_per_split;
    const int it1 = min(a.iters_total, it0 + a.iters_per_split);

    // ---- loader state: every thread keeps one fixed 8-channel column of each tile ---------------
    const int xcv = tid % XV, xrow = tid / XV;
    const int mrow0 = m0 + xcv * 8;
    const int tap = mrow0 / a.CP, xc0 = mrow0 - tap * a.CP;
    const int fr = tap / a.S, fs = tap - fr * a.S;
    const int x_nvalid = (tap < a.RS) ? a.C - xc0 : 0;
    const int ycv = tid % YV, yrow = tid / YV;
    const int yk0 = n0 + ycv * 8;
    const int y_nvalid = a.K - yk0;

    const Mask8 xmask = make_mask8(x_nvalid), ymask = make_mask8(y_nvalid);
    uint4 rx[XP], ry[YP];
    bool okx[XP], oky[YP];
    auto gload = [&](int it) {
        const int pbase = it * BK;
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            const int pix = pbase + xrow + i * XR;
            const uint32_t row = fdiv((uint32_t)pix, a.sQ);
            const int q = pix - (int)row * (int)a.sQ.d;
            const uint32_t n = fdiv(row, a.sP);
            const int p = (int)row - (int)n * (int)a.sP.d;
            const int ih = p * a.stride_h - a.pad_h + fr, iw = q * a.stride_w - a.pad_w + fs;
            okx[i] = pix < a.pixels && x_nvalid > 0 && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            const uint32_t off = (uint32_t)(((int)n * a.H + ih) * a.W + iw) * (uint32_t)a.xpitch + (uint32_t)xc0;
            rx[i] = ldg8<VEC>(a.X, okx[i] ? off : 0u, x_nvalid);
        }
#pragma unroll
        for (int i = 0; i < YP; ++i) {
            const int pix = pbase + yrow + i * YR;
            oky[i] = pix < a.pixels && y_nvalid > 0;
            ry[i] = ldg8<VEC>(a.DY, oky[i] ? (uint32_t)pix * (uint32_t)a.ypitch + (uint32_t)yk0 : 0u, y_nvalid);
        }
    };
    auto sstore = [&](int buf) {
        uint16_t* sX = smem + buf * STAGE_ELEMS;
        uint16_t* sY = sX + BK * LDM;
#pragma unroll
        for (int i = 0; i < XP; ++i)
            *reinterpret_cast<uint4*>(&sX[(xrow + i * XR) * LDM + xcv * 8]) = mask8(rx[i], okx[i], xmask);
#pragma unroll
        for (int i = 0; i < YP; ++i)
            *reinterpret_cast<uint4*>(&sY[(yrow + i * YR) * LDN + ycv * 8]) = mask8(ry[i], oky[i], ymask);
    };

    // ---- MFMA state ---------------------------------------------------------------------------
    const int wm = wave % WGM, wn = wave / WGM;
    // transpose-read geometry: 16-lane group g, lane t in group; source lane t points at pixel row
    // (t/4) and channel quad (t%4); the result is 4 consecutive pixels for channel 16*(g&1) + t.
    const int g16 = lane >> 4, t16 = lane & 15;
    const int tr_row = (g16 >> 1) * 8 + (t16 >> 2);     // + 4*h + ks*16
    const int tr_col = (g16 & 1) * 16 + (t16 & 3) * 4;  // + block origin
    f32x16 acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;
    bool m_live[TM], n_live[TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) m_live[tm] = m0 + wm * WTM + tm * 32 < a.Mtot;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) n_live[tn] = n0 + wn * WTN + tn * 32 < a.K;

    auto tr_read = [&](const uint16_t* base, int ld, int row, int col) -> bf16x8 {
        typedef __attribute__((address_space(3))) s16x4* lds_p;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(base + row * ld + col));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(base + (row + 4) * ld + col));
        s16x8 r;
        r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
        r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
        return __builtin_bit_cast(bf16x8, r);
    };

    if (it0 < it1) {
        gload(it0);
        sstore(0);
    }
    __syncthreads();
    bool all_live = true;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) all_live = all_live && m_live[tm];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) all_live = all_live && n_live[tn];
    auto compute = [&](int buf, auto check_tag) {
        constexpr bool CHECK = decltype(check_tag)::value;
        const uint16_t* sX = smem + buf * STAGE_ELEMS;
        const uint16_t* sY = sX + BK * LDM;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8 fx[TM], fy[TN];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) fx[tm] = tr_read(sX, LDM, ks * 16 + tr_row, wm * WTM + tm * 32 + tr_col);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) fy[tn] = tr_read(sY, LDN, ks * 16 + tr_row, wn * WTN + tn * 32 + tr_col);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    if (!CHECK || (m_live[tm] && n_live[tn]))
                        acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[tm], fy[tn], acc[tm][tn], 0, 0, 0);
        }
    };
    auto main_loop = [&](auto check_tag) {
        for (int it = it0; it < it1; ++it) {
            const int buf = (it - it0) & 1;
            if (it + 1 < it1) gload(it + 1);
            compute(buf, check_tag);
            if (it + 1 < it1) sstore(buf ^ 1);
            __syncthreads();
        }
    };
    if (all_live) main_loop(std::false_type{});
    else main_loop(std::true_type{});

    // ---- epilogue: lane holds k (column) = lane%32 and rows 8g + 4*(lane/32) + {0..3} = 4 consecutive c
    float* out = a.OUT + (a.direct ? 0 : (int64_t)split * a.K * a.out_row_pitch);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int k = n0 + wn * WTN + tn * 32 + (lane & 31);
        if (k >= a.K) continue;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int mrow = m0 + wm * WTM + tm * 32 + 8 * g + (lane >> 5) * 4;
                if (mrow >= a.Mtot) continue;
                const float v0 = acc[tm][tn][4 * g + 0], v1 = acc[tm][tn][4 * g + 1];
                const float v2 = acc[tm][tn][4 * g + 2], v3 = acc[tm][tn][4 * g + 3];
                if (a.direct) {
                    const int tp = mrow / a.CP, c = mrow - tp * a.CP;  // 4 consecutive rows share a tap (CP % 8 == 0)
                    float* dst = out + ((int64_t)k * a.RS + tp) * a.wpitch + c;
                    if (a.o_vec && c + 3 < a.C) {
                        *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
                    } else {
                        if (c < a.C) dst[0] = v0;
                        if (c + 1 < a.C) dst[1] = v1;
                        if (c + 2 < a.C) dst[2] = v2;
                        if (c + 3 < a.C) dst[3] = v3;
                    }
                } else {
                    *reinterpret_cast<float4*>(out + (int64_t)k * a.out_row_pitch + mrow) = make_float4(v0, v1, v2, v3);
                }
            }
        }
    }
}

template <int BM, int BN, int BK, int WGM, int WGN, int MINB, bool VEC = true>
inline hipError_t launch_wgrad_cfg(WgradArgs& a, hipStream_t st) {
    constexpr int NT = 64 * WGM * WGN;
    constexpr size_t lds = (size_t)2 * BK * (BM + 32 + BN + 32) * 2;
    auto kern = k_wgrad<BM, BN, BK, WGM, WGN, MINB, VEC>;
    static LdsOptIn opt_in;
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void*>(kern), lds); e != hipSuccess) return e;
    a.tiles_m = (int)ceil_div(a.Mtot, BM);
    a.tiles_n = (int)ceil_div(a.K, BN);
    hipLaunchKernelGGL(kern, dim3(a.tiles_m * a.tiles_n * a.splits), dim3(NT), lds, st, a);
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------- //
// weight gradient with direct global->LDS loads (vector path)
// ------------------------------------------------------------------------------------------- //
// Output tile: BM input channels of ONE filter tap x BN output channels; reduction over output pixels
// in steps of BKP.  Both tiles are pixel-major in LDS exactly as they sit in memory (a pixel row of
// the x tile is BM channels = 2*BM bytes), filled by 16-byte global->LDS loads and read back with the
// transpose read.  The 32-byte units of a row are permuted with the pixel row (see unit_phys in the kernel) so that
// the eight units the first and the second half-wave touch in one transpose read fall into different banks.  Pixels
// whose tap falls outside the image, and pixels past the end, are fetched as zeros (an out-of-range buffer offset, or
// the zero page in the general gather; both operands, so no garbage ever meets a zero).  Channel chunks past the channel count re-read the last valid chunk:
// they only feed accumulator rows/columns that are never stored.
// Transposing LDS read issued as inline assembly.  The compiler cannot see which LDS bytes the intrinsic
// form touches and therefore waits for every outstanding global->LDS load before it, which serialises the
// software pipeline; issued this way the read is ordered only by the explicit waits below.  The result
// registers must not be touched before lds_wait() has been applied to them.
template <int OFF>
__device__ __forceinline__ s16x4 lds_read_tr16_b64(uint32_t addr) {
    static_assert(OFF >= 0 && OFF < 65536, "DS offset field");
    s16x4 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
__device__ __forceinline__ bf16x8 join_halves(s16x4 lo, s16x4 hi) {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// KSPLIT wave groups share one tile: group g multiplies the g-th part of every stage's pixel sub-steps, and the
// groups' accumulators are added through LDS before the store.  More waves per SIMD to hide LDS and barrier
// latency, with the same LDS footprint, loads and partial-sum traffic as one group.
// XMODE: how x is addressed.  0 = any geometry (per-lane global addresses, advanced incrementally); 1 = stride 1 with
// an output grid equal to the input grid ('same'-padded filters): buffer loads whose moving part is a scalar; 2 = the
// same where no tap ever leaves the image (1 x 1 filters): no per-lane work at all in a reduction step.
// Operand loads stay in the caches, where the other tiles' workgroups find them: with the non-temporal hint on x, on dy, on
// both the train step of ResNet-50 is 3.5, 6, 8 % slower.
// `lin`: which workgroup of the problem this is, in split-major (split, tile) order.
template <int BM, int BN, int BKP, int WGM, int WGN, int STAGES, int KSPLIT, int XMODE, bool AHEAD>
__device__ __forceinline__ void wgrad_dl_body(const WgradArgs& a, const int lin, uint8_t* smem_b) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
    constexpr int NWT = WGM * WGN;       // waves of one group: the wave grid over the tile
    constexpr int NW = NWT * KSPLIT;     // all waves: they share the loads
    constexpr int RBX = BM * 2, RBY = BN * 2;              // bytes per pixel row
    constexpr int CPRX = RBX / 16, CPRY = RBY / 16;        // 16-byte chunks per row
    constexpr int RPLX = 64 / CPRX, RPLY = 64 / CPRY;      // pixel rows per wave-level load
    constexpr int LX = BKP / RPLX / NW, LY = BKP / RPLY / NW;  // loads per lane per stage
    constexpr int LPT = LX + LY;
    constexpr int XBYTES = BKP * RBX, STAGE_BYTES = BKP * (RBX + RBY);
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    static_assert((RBX == 128 || RBX == 256) && (RBY == 128 || RBY == 256), "row size");
    static_assert(NW % 2 == 0 && LX >= 1 && LY >= 1 && BKP % (RPLX * NW) == 0 && BKP % (RPLY * NW) == 0, "tile config");
    static_assert(TM >= 1 && TN >= 1 && BKP % 16 == 0 && STAGES >= 2 && (STAGES - 2) * LPT < 64, "tile config");
    static_assert(KSPLIT >= 1 && (BKP / 16) % KSPLIT == 0 && NW <= 16, "wave groups");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / NWT, wave_t = wave - kg * NWT;  // wave group, wave inside the group
    const int ntile = a.tiles_m * a.tiles_n;
    const int split = (int)fdiv((uint32_t)lin, a.ntile_div);
    const int tile = lin - split * ntile;
    const int mt = (int)fdiv((uint32_t)tile, a.tn_div);  // (tap, channel block)
    const int n0 = (tile - mt * a.tiles_n) * BN;   // k origin
    // tile row block: one filter tap (CP channels), or in folded mode one filter row (S*CP contiguous elements)
    const int tb = (int)fdiv((uint32_t)mt, a.tap_div);
    const int cb = (mt - tb * a.tiles_per_tap) * BM;
    const int run = a.fold ? a.S * a.CP : a.CP;
    const int fr = a.fold ? tb : (int)fdiv((uint32_t)tb, a.S_div);
    const int it0 = split * a.iters_per_split;
    const int it1 = min(a.iters_total, it0 + a.iters_per_split);

    // Placement of the 32-byte units (16 channels) of a pixel row, constant per lane over its loads.  A transposing
    // read takes, per 16-lane group, one unit from each of four consecutive pixel rows, and the LDS serves two such
    // groups per cycle (64 banks of 4 bytes): lanes 0-31 read units u and u + 1 (u even) of the same four rows, lanes
    // 32-63 the same of rows + 8.  So the low bit of the logical unit becomes the high bit of the physical one (u and
    // u + 1 land in different halves of a 256-byte bank line) and the remaining bits are XOR-ed with the row so that
    // the four rows of a group differ: 2.5 instead of 4.1 cycles per read against XOR-ing all bits with the row.
    // 128-byte rows: consecutive rows already alternate between the halves of a bank line.
    auto unit_phys = [](int u, int row, int rb) {
        return rb == 256 ? (((u >> 1) | ((u & 1) << 2)) ^ (row & 3)) : ((((u & 1) << 1) | (u >> 1)) ^ ((row >> 1) & 1));
    };
    auto unit_logical = [](int p, int row, int rb) {  // inverse of unit_phys in u
        if (rb == 256) {
            const int q = p ^ (row & 3);
            return ((q & 3) << 1) | (q >> 2);
        }
        const int q = p ^ ((row >> 1) & 1);
        return ((q & 1) << 1) | (q >> 1);
    };
    // x tile: this lane's row inside a wave-level load, and the logical 8-channel chunk it fetches
    const int xr = lane / CPRX, xpc = lane % CPRX;
    const int xlc = (unit_logical(xpc >> 1, wave * RPLX + xr, RBX) << 1) | (xpc & 1);
    const int xc = min(cb + xlc * 8, run - 8);     // clamp: chunks past the run are never stored
    const int fs = a.fold ? (int)fdiv((uint32_t)xc, a.CP_div) : tb - fr * a.S;   // filter column of this lane's chunk
    const int fs_addr = a.fold ? 0 : fs;           // folded: the column offset is part of xc
    const int yr = lane / CPRY, ypc = lane % CPRY;
    const int ylc = (unit_logical(ypc >> 1, wave * RPLY + yr, RBY) << 1) | (ypc & 1);
    const int yk = min(n0 + ylc * 8, a.KP - 8);
    const uint16_t* zero_page = reinterpret_cast<const uint16_t*>(g_zero16);

    // Gather state of this lane's loads, advanced by BKP pixels per reduction step without divisions or multiplies
    // (integer multiplies run at a quarter of the vector rate and were the loop's bound).  A step moves every
    // slot from output pixel (n, p, q) to (n + dn, p + dp, q + dq) with at most one carry out of q and one out of
    // p (dq < Q, dp < P); the slot keeps the input coordinates (ih, iw) of its tap and the element offset of that
    // input pixel, which change by constants that depend only on the two carries.
    const int Qs = (int)a.Q.d * a.stride_w, Ps = (int)a.P.d * a.stride_h;
    const int iw_wrap = Qs - a.pad_w + fs, ih_wrap = Ps - a.pad_h + fr;  // first coordinate past the last output column / row
    const int dq_s = a.dq * a.stride_w, dp_s = a.dp * a.stride_h;
    const int rowp = a.W * a.xpitch;  // elements per input row
    const int D0 = dq_s * a.xpitch + dp_s * rowp + a.dn * a.H * rowp;  // no carry
    const int D1 = a.stride_h * rowp - Qs * a.xpitch;                  // carry out of q: next output row
    const int D2 = (a.H - Ps) * rowp;                                  // carry out of p: next image
    const int xrel0 = wave * RPLX + xr, yrel0 = wave * RPLY + yr;      // this lane's pixel inside a step (slot 0)
    [[maybe_unused]] int x_ih[LX], x_iw[LX];
    [[maybe_unused]] uint32_t x_off[LX];
    // XMODE 1 needs only whether the tap is inside the image: the pixel's place in its row and in its image, both counted
    // cyclically from the first pixel for which it is, is below the number of those.  Two counters without a carry between
    // them, an addition, a subtraction and an unsigned minimum a step each (what lies below zero is large).
    [[maybe_unused]] const int Qd = (int)a.Q.d, PQ = Qd * (int)a.P.d;
    [[maybe_unused]] const int q_lo = max(0, a.pad_w - fs), m_lo = max(0, a.pad_h - fr) * Qd;
    [[maybe_unused]] const uint32_t q_n = (uint32_t)max(0, min(Qd, a.W + a.pad_w - fs) - q_lo);
    [[maybe_unused]] const uint32_t m_n = (uint32_t)max(0, min((int)a.P.d, a.H + a.pad_h - fr) * Qd - m_lo);
    [[maybe_unused]] const uint32_t q_step = (uint32_t)a.dq, m_step = (uint32_t)(a.dp * Qd + a.dq);  // BKP modulo Qd and PQ
    [[maybe_unused]] uint32_t x_q[LX], x_m[LX];
    if constexpr (XMODE < 2) {
#pragma unroll
        for (int j = 0; j < LX; ++j) {
            const int pix = it0 * BKP + xrel0 + NW * j * RPLX;
            const uint32_t row = fdiv((uint32_t)pix, a.Q);
            const int q = pix - (int)row * (int)a.Q.d;
            const uint32_t n = fdiv(row, a.P);
            const int p = (int)row - (int)n * (int)a.P.d;
            if constexpr (XMODE == 0) {
                x_ih[j] = p * a.stride_h - a.pad_h + fr;
                x_iw[j] = q * a.stride_w - a.pad_w + fs;
                x_off[j] = (uint32_t)(((int)n * a.H + x_ih[j]) * a.W + (x_iw[j] - fs + fs_addr)) * (uint32_t)a.xpitch + (uint32_t)xc;
            } else {
                const int m = p * Qd + q;
                x_q[j] = (uint32_t)(q >= q_lo ? q - q_lo : q - q_lo + Qd);
                x_m[j] = (uint32_t)(m >= m_lo ? m - m_lo : m - m_lo + PQ);
            }
        }
    }
    // pixels from the next step's first one to the end of this workgroup's slice (uniform): loads past it fetch zeros,
    // so steps may be issued unconditionally
    int p_left = min(a.pixels, it1 * BKP) - it0 * BKP;

    // dy, and x in layers whose output grid equals the input grid at stride 1 (1x1 and 'same'-padded filters), sit at
    // an address that is affine in the output pixel index: a reduction step moves every load by one uniform amount.
    // Those loads are buffer loads: the per-lane part of the address is a constant (voffset), the moving part a
    // scalar register (soffset), and a lane that must read zeros (tap outside the image, pixel past the end) passes
    // an out-of-range voffset, for which the load writes zeros to LDS.  The loop is bound by the number of
    // instructions a wave issues per step, so nothing is computed per lane and step beyond the validity of
    // 'same'-padded taps.  The filter tap's shift is folded into the buffer's base address (it may point ahead of the
    // tensor: only valid taps are ever fetched).
    constexpr uint32_t kBufRecords = 0x40000000u, kBufOut = 0x80000000u, kBufFlags = 0x00020000u;
    const int tapshift = XMODE ? ((fr - a.pad_h) * a.W + (fs_addr - a.pad_w)) * a.xpitch : 0;  // uniform
    const __amdgpu_buffer_rsrc_t x_srd =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.X) + tapshift, 0, kBufRecords, kBufFlags);
    const __amdgpu_buffer_rsrc_t y_srd = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.DY), 0, kBufRecords, kBufFlags);
    const uint32_t x_v = (uint32_t)(xr * a.xpitch + xc) * 2u, y_v = (uint32_t)(yr * a.ypitch + yk) * 2u;  // bytes
    uint32_t x_s[LX], y_s[LY];  // scalar byte offsets of the slots' pixel rows
#pragma unroll
    for (int j = 0; j < LX; ++j) x_s[j] = (uint32_t)(it0 * BKP + (wave + NW * j) * RPLX) * (uint32_t)a.xpitch * 2u;
#pragma unroll
    for (int j = 0; j < LY; ++j) y_s[j] = (uint32_t)(it0 * BKP + (wave + NW * j) * RPLY) * (uint32_t)a.ypitch * 2u;
    const uint32_t x_step = (uint32_t)(BKP * a.xpitch) * 2u, y_step = (uint32_t)(BKP * a.ypitch) * 2u;

    // issue the loads of the next reduction step (steps are issued in order, x before dy) into `stage`
    auto issue_x = [&](int stage) {
        uint8_t* sbase = smem_b + stage * STAGE_BYTES;
        const bool whole = p_left >= BKP;  // uniform: every pixel of the step lies inside the slice
        if constexpr (XMODE == 0) {
#pragma unroll
            for (int j = 0; j < LX; ++j) {
                const bool ok = xrel0 < p_left - NW * j * RPLX && (unsigned)x_ih[j] < (unsigned)a.H && (unsigned)x_iw[j] < (unsigned)a.W;
                __builtin_amdgcn_global_load_lds(pick_ptr(ok, a.X + x_off[j], zero_page),
                                                 (lds_void_ptr)(sbase + (wave + NW * j) * 1024), 16, 0, 0);
                const int iw = x_iw[j] + dq_s;
                const bool c1 = iw >= iw_wrap;
                x_iw[j] = iw - (c1 ? Qs : 0);
                const int ih = x_ih[j] + (c1 ? dp_s + a.stride_h : dp_s);
                const bool c2 = ih >= ih_wrap;
                x_ih[j] = ih - (c2 ? Ps : 0);
                x_off[j] += (uint32_t)((c1 ? D0 + D1 : D0) + (c2 ? D2 : 0));
            }
        } else {
            uint32_t v[LX];
#pragma unroll
            for (int j = 0; j < LX; ++j) {
                v[j] = x_v;
                if constexpr (XMODE == 1) {
                    v[j] = x_q[j] < q_n && x_m[j] < m_n ? x_v : kBufOut;
                    x_q[j] = min(x_q[j] + q_step, x_q[j] + (q_step - (uint32_t)Qd));
                    x_m[j] = min(x_m[j] + m_step, x_m[j] + (m_step - (uint32_t)PQ));
                }
            }
            if (!whole) {
#pragma unroll
                for (int j = 0; j < LX; ++j) v[j] = xrel0 < p_left - NW * j * RPLX ? v[j] : kBufOut;
            }
#pragma unroll
            for (int j = 0; j < LX; ++j) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(x_srd, (lds_void_ptr)(sbase + (wave + NW * j) * 1024), 16, v[j], x_s[j], 0, 0);
                x_s[j] += x_step;
            }
        }
    };
    auto issue_y = [&](int stage) {
        uint8_t* sbase = smem_b + stage * STAGE_BYTES;
        uint32_t vy[LY];
#pragma unroll
        for (int j = 0; j < LY; ++j) vy[j] = y_v;
        if (p_left < BKP) {
#pragma unroll
            for (int j = 0; j < LY; ++j) vy[j] = yrel0 < p_left - NW * j * RPLY ? y_v : kBufOut;
        }
#pragma unroll
        for (int j = 0; j < LY; ++j) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(y_srd, (lds_void_ptr)(sbase + XBYTES + (wave + NW * j) * 1024), 16, vy[j], y_s[j], 0, 0);
            y_s[j] += y_step;
        }
        p_left -= BKP;
    };

    // ---- MFMA state ---------------------------------------------------------------------------
    const int wm = wave_t % WGM, wn = wave_t / WGM;
    // transpose-read geometry: 16-lane group g16, lane t16; source lane t16 points at pixel row (t16 >> 2)
    // and channel quad (t16 & 3); the result is 4 consecutive pixels for channel 16*(g16 & 1) + t16.
    const int g16 = lane >> 4, t16 = lane & 15;
    const int tr_row = (g16 >> 1) * 8 + (t16 >> 2);  // + 4*h + ks*16
    const int tr_u = (g16 & 1);                       // 16-channel unit inside a 32-channel block
    const int tr_b = (t16 & 3) * 8;                   // byte inside the unit
    f32x16 acc[TM][TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.f;

    // 32-bit LDS addresses of this lane's transposing reads: per 32-wide tile the 4-pixel halves at rows r, r+4.
    // The swizzle term does not depend on the 16-pixel sub-step, which therefore is an immediate offset.
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem_b;
    constexpr int NKS = BKP / 16 / KSPLIT, NRD = 2 * (TM + TN);  // sub-steps per stage and group, LDS reads per sub-step
    uint32_t ax[TM][2], ay[TN][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = tr_row + 4 * h;
        const int r0 = kg * NKS * 16;  // first pixel row of this group's sub-steps (a multiple of 16: same swizzle)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int u = (wm * WTM + tm * 32) / 16 + tr_u;
            ax[tm][h] = lds_base + (uint32_t)((r0 + r) * RBX + (unit_phys(u, r, RBX) << 5) + tr_b);
        }
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int u = (wn * WTN + tn * 32) / 16 + tr_u;
            ay[tn][h] = lds_base + (uint32_t)((r0 + r) * RBY + (unit_phys(u, r, RBY) << 5) + tr_b);
        }
    }
    static_assert(NKS == 1 || NRD < 16, "fragment reads per sub-step must fit the lgkmcnt field");
    static_assert(NKS % 2 == 0, "fragment buffers alternate between sub-steps");
    s16x4 fx[2][TM][2], fy[2][TN][2];
    auto issue_reads = [&](auto ks_c, uint32_t sb) {
        constexpr int KS = decltype(ks_c)::value;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int h = 0; h < 2; ++h) fx[KS & 1][tm][h] = lds_read_tr16_b64<KS * 16 * RBX>(ax[tm][h] + sb);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int h = 0; h < 2; ++h) fy[KS & 1][tn][h] = lds_read_tr16_b64<XBYTES + KS * 16 * RBY>(ay[tn][h] + sb);
    };
    // PENDING: reads issued after those of this sub-step, which may stay in flight
    auto multiply = [&](auto b_c, auto pending_c) {
        constexpr int B = decltype(b_c)::value;
        lds_wait<decltype(pending_c)::value>(fx[B][0][0]);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int h = 0; h < 2; ++h) lds_tie(fx[B][tm][h]);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int h = 0; h < 2; ++h) lds_tie(fy[B][tn][h]);
        bf16x8 vx[TM], vy[TN];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) vx[tm] = join_halves(fx[B][tm][0], fx[B][tm][1]);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) vy[tn] = join_halves(fy[B][tn][0], fy[B][tn][1]);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vy[tn], vx[tm], acc[tm][tn], 0, 0, 0);
        // keep this sub-step's MFMAs ahead of what follows: otherwise the scheduler sinks them below the next wait and
        // nothing overlaps the fragment reads
        __builtin_amdgcn_sched_barrier(0);
    };
    typedef std::integral_constant<int, NRD> one_sub_step;
    typedef std::integral_constant<int, 0> none;

    const int nk = it1 - it0;
    constexpr bool TURNS = XMODE == 1 && AHEAD && KSPLIT > 1;  // (see the loop)
    [[maybe_unused]] const bool late = (wave & 4) != 0;  // waves w and w + 4 share a SIMD
    auto issue = [&](int stage) {
        issue_x(stage);
        issue_y(stage);
    };
    // Loads run STAGES - 1 steps ahead and are issued at every step, also past the slice's end (they then fetch
    // zeros into a stage nobody multiplies): the number of loads in flight is the same at every wait.
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue(s);
    if constexpr (AHEAD) {
        // Fragments are read two sub-steps ahead of their MFMAs, across the barrier between stages: sub-step ks of stage t
        // multiplies what was read during stage t - 1 and then reads sub-step ks of stage t + 1.  A read behind the barrier
        // that publishes its stage costs the LDS latency once a stage (256 -> 256 channels at 14 x 14, 64 more images:
        // 16.0 -> 14.8 us).  The price is one more stage, since a stage is published one step before it is multiplied.
        static_assert(STAGES >= 3, "stages");
        wait_vmcnt<(STAGES - 2) * LPT>();
        barrier_nofence();
        issue_reads(std::integral_constant<int, 0>{}, 0u);
        issue_reads(std::integral_constant<int, 1>{}, 0u);
    }
    for (int kt0 = 0; kt0 < nk; kt0 += STAGES) {
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            if (kt0 + s < nk) {
                if constexpr (AHEAD) wait_vmcnt<(STAGES - 3) * LPT>();  // the next stage has landed ...
                else wait_vmcnt<(STAGES - 2) * LPT>();                  // this stage has landed ...
                barrier_nofence();  // ... for every wave, and nobody reads the previous one any more
                // A later step's loads go out between this step's MFMAs, x behind the first sub-step's and dy behind the last's,
                // into the buffer consumed in the previous step.  A CU's address unit takes 16 clocks for each of a step's 16
                // to 24 load instructions, which then do not hold up the fragment reads of the waves that come after: 14 x 14, 256 -> 256,
                // 3 x 3, alone, against all loads ahead of the MFMAs in one of the two waves of a SIMD and behind them in the other
                // 22.0 -> 21.0 us, 7 x 7, 512 -> 512 30.3 -> 28.8.  With two wave groups the turns of the waves stay the better order for
                // XMODE 1 alone on the chip (7 x 7, 239 -> 383: 17.4 and 17.6 us).  (All loads behind the MFMAs in every wave: 7 % longer.)
                const int to = (s + STAGES - 1) % STAGES;
                if constexpr (TURNS) {
                    if (!late) issue(to);
                }
                const uint32_t cur = (uint32_t)(s * STAGE_BYTES), nxt = (uint32_t)(((s + 1) % STAGES) * STAGE_BYTES);
                if constexpr (!AHEAD) issue_reads(std::integral_constant<int, 0>{}, cur);
                static_for<0, NKS>([&](auto ks_c) {
                    constexpr int KS = decltype(ks_c)::value;
                    typedef std::integral_constant<int, (KS & 1)> buf;
                    if constexpr (AHEAD) {
                        multiply(buf{}, one_sub_step{});
                        if constexpr (KS + 2 < NKS) issue_reads(std::integral_constant<int, KS + 2>{}, cur);
                        else issue_reads(std::integral_constant<int, KS + 2 - NKS>{}, nxt);
                    } else if constexpr (KS + 1 < NKS) {  // the next sub-step's reads are in flight while this one multiplies
                        issue_reads(std::integral_constant<int, KS + 1>{}, cur);
                        multiply(buf{}, one_sub_step{});
                    } else {
                        multiply(buf{}, none{});
                    }
                    if constexpr (KS == 0 && !TURNS) issue_x(to);
                });
                if constexpr (!TURNS) issue_y(to);
                else if (late) issue(to);
            }
        }
    }
    if constexpr (AHEAD) {  // the fragments of the step past the end
        lds_wait<0>(fx[0][0][0]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) lds_tie(fx[i >> 1][tm][i & 1]);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) lds_tie(fy[i >> 1][tn][i & 1]);
        }
    }
    wait_vmcnt<0>();  // the loads issued past the end have landed before LDS is reused or the wave ends

    if constexpr (KSPLIT > 1) {
        // groups 1.. park their accumulators in LDS one group at a time (the stage buffers are dead: every load was
        // waited for and the barrier below follows every wave's last read); group 0 adds them in group order and stores
        float* red = reinterpret_cast<float*>(smem_b);
        constexpr int PER_WAVE = TM * TN * 16 * 64;
#pragma unroll
        for (int g = 1; g < KSPLIT; ++g) {
            __syncthreads();
            if (kg == g) {
                float* dst = red + wave_t * PER_WAVE + lane;
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                        for (int v = 0; v < 16; ++v) dst[((tm * TN + tn) * 16 + v) * 64] = acc[tm][tn][v];
            }
            __syncthreads();
            if (kg == 0) {
                const float* src = red + wave_t * PER_WAVE + lane;
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[tm][tn][v] += src[((tm * TN + tn) * 16 + v) * 64];
            }
        }
        if (kg > 0) return;
    }
    // ---- epilogue: the MFMA's row operand is dy, so a lane holds input channel (column) lane%32 of the 32x32 block
    // and output channels (rows) 8g + 4*(lane/32) + {0..3}: a store instruction writes, for one output channel per
    // half-wave, 32 consecutive input channels = 128 contiguous bytes of dw (or of the partial slab).
    // Buffer stores on a descriptor of the tile's rows: 32-bit offsets, and what must not be written (output channels past
    // the last one, input channels past the run) is out of range, so the 16 * TM * TN stores are that many instructions and
    // an addition each (1.75 us of a workgroup's life with a 64-bit address and a branch per store, 0.8 us so).
    const int row_pitch = a.direct ? a.RS * a.wpitch : a.out_row_pitch, tap_pitch = a.direct ? a.wpitch : a.CP;
    const int64_t first = (int64_t)n0 * row_pitch + (a.direct ? 0 : (int64_t)split * a.K * a.out_row_pitch);
    const uint32_t tile_bytes = (uint32_t)(min(a.K - n0, BN) * row_pitch) * 4u;  // <= 2^31 (plan_wgrad_tiles)
    const __amdgpu_buffer_rsrc_t o_srd = __builtin_amdgcn_make_buffer_rsrc(a.OUT + first, 0, tile_bytes, kBufFlags);
    const int cols = a.direct ? a.C : a.CP, row0 = wn * WTN + (lane >> 5) * 4;  // output channel of element (tn, e) = (0, 0)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int cr = cb + wm * WTM + tm * 32 + (lane & 31);  // row inside the run
        const int ts = a.fold ? (int)fdiv((uint32_t)cr, a.CP_div) : 0;
        const int c = cr - ts * a.CP;
        const int tapi = a.fold ? tb * a.S + ts : tb;
        const bool ok = cr < run && c < cols;
        const uint32_t at0 = ok ? (uint32_t)(row0 * row_pitch + tapi * tap_pitch + c) * 4u : kBufOut;
        auto at = [&](int tn, int e) { return at0 + (uint32_t)((tn * 32 + 8 * (e >> 2) + (e & 3)) * row_pitch) * 4u; };
        if (a.direct && a.lw) {  // uniform: regulariser folded in
            // every weight and norm this lane needs is fetched before the first store: the stores may alias the loads
            // as far as the compiler knows, and interleaved they would each wait out a full memory round trip
            const __amdgpu_buffer_rsrc_t w_srd =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.lw) + first, 0, tile_bytes, kBufFlags);
            const float in = a.l_in && ok ? a.l_in[c] : 0.f;
            const float inv_in = in > 0.f ? 1.0f / in : 0.f;
            float wv[TN][16], io[TN][16];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    wv[tn][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(w_srd, at(tn, e), 0, 0));
                    io[tn][e] = a.l_on ? a.l_on[min(n0 + row0 + tn * 32 + 8 * (e >> 2) + (e & 3), a.K - 1)] : 0.f;
                }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float inv_out = io[tn][e] > 0.f ? 1.0f / io[tn][e] : 0.f;
                    const float v = acc[tm][tn][e] + a.l_lambda * (wv[tn][e] * (inv_out + inv_in));
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), o_srd, at(tn, e), 0, 0);
                }
            continue;
        }
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[tm][tn][e]), o_srd, at(tn, e), 0, 0);
    }
#endif
}

// ------------------------------------------------------------------------------------------- //
// weight gradient of 3 x 3 filters at stride 1 and padding 1: the three taps of a filter row from one tile of x
// ------------------------------------------------------------------------------------------- //
// What bounds wgrad_dl_body on these layers is the way of the operands into LDS (64 bytes a clock and CU) and out of it
// again, one after the other: a 128 x 128 tile takes 16 KB in and 48 KB out for 32 pixels, 0.22 to 0.28 us where its MFMAs
// are 0.11, whatever the number of stages.  Here a workgroup owns one filter row (three taps) x 64 input channels x 64 output
// channels: 12288 outputs for the operand bytes of a 64 x 64 tile.  The taps of a row read the same pixels one place
// further, so they are three windows of the same LDS rows; what keeps a window from running into the next image row is a
// column of zeros behind every one.  The reduction therefore counts W + 1 places a row ("positions"; 1 / W more of them), and both
// operands hold zeros there.  Which image row a tap needs is the same for the whole workgroup: x is fetched shifted, rows
// outside the image as zeros.
//   Eight waves: two halves of the input channels x four of a step's 64 positions.  A wave multiplies 16 positions a step
// (3 x fragments and 2 dy fragments for 6 MFMAs), its fragments read a step ahead; the four position groups are added
// through LDS at the end, in a fixed order, tap by tap, by all threads (2 us with the set-up: calls of few steps stay with the
// other forms).  A step of 64 positions is 0.28 us with operands from memory (17 KB in at some 70 bytes a ns, which is what a CU
// gets of lines that no other has fetched before; 0.16 us without the loads, its MFMAs).  Main kernel, 64 images, 240 to 252
// workgroups, from memory: 14 x 14, 256 -> 256 23.5 -> 21.3 us, 28 x 28, 128 -> 128 22.9 -> 21.8, 56 x 56, 64 -> 64 34.9 -> 23.1;
// with 64 x 64 tiles 252 workgroups fetch 462 MB for the last, so 157.  Whole calls 26.6 -> 26.1, 26.1 -> 25.7, 29.7 -> 24.6, 7 x 7,
// 512 -> 512 30.2 -> 25.7, 30 x 14 x 14, 512 -> 512 50.6 -> 39.0; training step of ResNet-50 3255 -> 3186 us, pruned 2679 -> 2638.
// Five stages: four 1 to 2 us longer, six and eight the same.
//   A place of the zero column multiplies a zero of dy with the x beside it, which is no tap's: an infinity or a NaN there
// would reach taps that never read it.  Such a product is a NaN, and so is the tap's sum: a workgroup that finds one in its
// outer taps runs its slice again with x cleared at those places (MASKED), so that only what a tap reads can make its
// sum one.  The look for a NaN costs 0.2 to 0.4 us of a call's 26 (once a slice; 40 us calls beside others 0.4).  (The other way
// round, a dy that is not finite meets a zero of x outside the image, here as in wgrad_dl_body.)
// A workgroup's slice in positions; a.Q.d is W + 1 and a.pixels the number of positions.  Offsets inside a slice in 24 bits times a
// pitch, below kBufRecords (wgrad_row3_ok).
constexpr int kRow3Px = 64;
constexpr int kRow3XBytes = (kRow3Px / 8 + 1) * 1024;  // 66 rows of 64 channels, in loads of eight rows
constexpr int kRow3StageBytes = kRow3XBytes + kRow3Px * 128;
constexpr int kRow3ReduceBytes = 64 * 1024;
// Returns whether the slice is to be run again.
template <int STAGES, bool MASKED>
__device__ __forceinline__ bool wgrad_row3_body(const WgradArgs& a, const int lin, uint8_t* smem_b) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
    static_assert(STAGES >= 4 && STAGES * kRow3StageBytes >= kRow3ReduceBytes + 8 * 4 && STAGES * kRow3StageBytes <= 160 * 1024, "LDS");
    constexpr uint32_t kBufRecords = 0x40000000u, kBufOut = 0x80000000u, kBufFlags = 0x00020000u;
    int lane = threadIdx.x & 63;
    if constexpr (MASKED) asm volatile("" : "+v"(lane));  // (nothing of the first run is kept in registers for this one)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wc = wave & 1, wp = wave >> 1;  // half of the input channels, quarter of a step's positions
    const int split = (int)fdiv((uint32_t)lin, a.ntile_div);
    const int tile = lin - split * (a.tiles_m * a.tiles_n);
    const int mt = (int)fdiv((uint32_t)tile, a.tn_div);
    const int n0 = (tile - mt * a.tiles_n) * 64;
    const int fr = (int)fdiv((uint32_t)mt, a.tap_div);  // filter row
    const int cb = (mt - fr * a.tiles_per_tap) * 64;
    const int it0 = split * a.iters_per_split;
    const int it1 = min(a.iters_total, it0 + a.iters_per_split);
    const int nk = it1 - it0;

    // ---- loads: a wave fetches eight positions of either operand a step, wave 0 also the two of x behind the step's last one.
    // Row i of the x tile is position (start - 1 + i), row i of the dy tile position (start + i).
    // (placement of the 32-byte units as in wgrad_dl_body, 128-byte rows)
    const int lr = lane >> 3, row = wave * 8 + lr;
    const int up = ((lane & 7) >> 1) ^ ((lr >> 1) & 1), lc = ((((up & 1) << 1) | (up >> 1)) << 1) | (lane & 1);
    const uint32_t xcb = (uint32_t)min(cb + lc * 8, a.CP - 8) * 2u, ycb = (uint32_t)min(n0 + lc * 8, a.KP - 8) * 2u;
    const int Qp = (int)a.Q.d, PQ = Qp * (int)a.P.d;
    const int t0 = it0 * kRow3Px, t1 = min(a.pixels, it1 * kRow3Px);
    const int pix0 = t0 - (int)fdiv((uint32_t)t0, a.Q);  // pixel of the slice's first position
    // place in the row, place in the image counted cyclically from the first one whose tap row lies inside, pixel
    const int m_lo = fr == 0 ? Qp : 0;
    const uint32_t m_n = (uint32_t)(fr == 1 ? PQ : PQ - Qp);
    const uint32_t q_step = (uint32_t)a.dq, m_step = (uint32_t)(a.dp * Qp + a.dq);  // positions of a step modulo Qp and PQ
    const uint32_t p_step = (uint32_t)(kRow3Px - kRow3Px / Qp);
    uint32_t q, m, pix;
    {
        const int t = t0 + row;
        const uint32_t rw = fdiv((uint32_t)t, a.Q);
        const uint32_t n = fdiv(rw, a.P);
        q = (uint32_t)(t - (int)rw * Qp);
        const int mm = ((int)rw - (int)n * (int)a.P.d) * Qp + (int)q;
        m = (uint32_t)(mm >= m_lo ? mm - m_lo : mm - m_lo + PQ);
        pix = (uint32_t)(t - (int)rw - pix0);
    }
    // positions from the step's first one to the end: of the slice for dy, for x two further (but not past the last image)
    int y_left = t1 - t0, x_left = min(t1 + 2, a.pixels + 1) - t0;
    const uint32_t xpb = (uint32_t)a.xpitch * 2u, ypb = (uint32_t)a.ypitch * 2u;
    const __amdgpu_buffer_rsrc_t x_srd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(a.X) + ((int64_t)pix0 + (fr - 1) * a.W - 1) * a.xpitch, 0, kBufRecords, kBufFlags);
    const __amdgpu_buffer_rsrc_t y_srd =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.DY) + (int64_t)pix0 * a.ypitch, 0, kBufRecords, kBufFlags);
    typedef __attribute__((address_space(3))) uint8_t* lds_bytes;
    const lds_bytes x_to = (lds_bytes)smem_b + wave * 1024, y_to = x_to + kRow3XBytes, halo_to = (lds_bytes)smem_b + kRow3Px * 128;
    auto issue = [&](int stage) {
        const uint32_t ox = __umul24(pix, xpb) + xcb, oy = __umul24(pix, ypb) + ycb;
        const uint32_t vx = (q != 0) & (m < m_n) & (row < x_left) ? ox : kBufOut;
        const uint32_t vy = (q != (uint32_t)(Qp - 1)) & (row < y_left) ? oy : kBufOut;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(x_srd, (lds_void_ptr)(x_to + stage * kRow3StageBytes), 16, vx, 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(y_srd, (lds_void_ptr)(y_to + stage * kRow3StageBytes), 16, vy, 0, 0, 0);
        const uint32_t qs = q + q_step;
        pix += p_step;
        asm("" : "+v"(pix));  // (or the carry is subtracted from p_step first, an instruction more)
        pix -= qs >= (uint32_t)Qp ? 1u : 0u;
        q = min(qs, qs - (uint32_t)Qp);
        m = min(m + m_step, m + (m_step - (uint32_t)PQ));
        x_left -= kRow3Px;
        y_left -= kRow3Px;
        if (wave == 0) {  // (its first rows of the next step)
            const uint32_t oh = __umul24(pix, xpb) + xcb;
            const uint32_t vh = (lr < 2) & (q != 0) & (m < m_n) & (row < x_left) ? oh : kBufOut;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_srd, (lds_void_ptr)(halo_to + stage * kRow3StageBytes), 16, vh, 0, 0, 0);
        }
    };
    auto wait_stages = [&](auto n_c) {  // all but the loads of the last n steps have landed
        constexpr int N = decltype(n_c)::value;
        wait_vmcnt<3 * N>();
        if (wave != 0) wait_vmcnt<2 * N>();
    };

    // ---- fragments (transposing reads as in wgrad_dl_body; four rows further the placement is the same)
    const int g16 = lane >> 4, t16 = lane & 15;
    const int tr_row = wp * 16 + (g16 >> 1) * 8 + (t16 >> 2), tr_u = g16 & 1, tr_b = (t16 & 3) * 8;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem_b;
    auto frag_at = [&](int r, int block) {
        const int u = tr_u + 2 * block;
        return lds_base + (uint32_t)(r * 128 + ((((((u & 1) << 1) | (u >> 1)) ^ ((r >> 1) & 1))) << 5) + tr_b);
    };
    uint32_t ax[3], ay[2];
#pragma unroll
    for (int s = 0; s < 3; ++s) ax[s] = frag_at(tr_row + s, wc);
#pragma unroll
    for (int b = 0; b < 2; ++b) ay[b] = frag_at(tr_row, b) + kRow3XBytes;
    // MASKED: which of a lane's eight positions lie in the zero column (the places every W + 1 from there on are known as bits)
    [[maybe_unused]] uint32_t q_frag = 0, column = 0, zeros = 0;
    if constexpr (MASKED) {
        const uint32_t t = (uint32_t)(t0 + wp * 16 + (lane >> 5) * 8);
        q_frag = t - fdiv(t, a.Q) * (uint32_t)Qp;
        for (int b = 0; b < 8; b += Qp) column |= 1u << b;
    }
    f32x16 acc[3][2];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][b][v] = 0.f;
    s16x4 fx[3][2], fy[2][2][2];
    auto read_x = [&](auto s_c, uint32_t sb) {
        constexpr int S = decltype(s_c)::value;
        fx[S][0] = lds_read_tr16_b64<0>(ax[S] + sb);
        fx[S][1] = lds_read_tr16_b64<512>(ax[S] + sb);
    };
    auto read_y = [&](auto b_c, uint32_t sb) {
        constexpr int B = decltype(b_c)::value;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            fy[B][b][0] = lds_read_tr16_b64<0>(ay[b] + sb);
            fy[B][b][1] = lds_read_tr16_b64<512>(ay[b] + sb);
        }
    };
    // the eight reads behind the ones that tap S needs may stay in flight
    auto multiply = [&](auto s_c, auto b_c) {
        constexpr int S = decltype(s_c)::value, B = decltype(b_c)::value;
        lds_wait<8>(fx[S][0]);
        lds_tie(fx[S][1]);
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) lds_tie(fy[B][b][h]);
        bf16x8 vx = join_halves(fx[S][0], fx[S][1]);
        if constexpr (MASKED && S != 1) {  // (the middle tap reads the zero column there)
            u32x4 w = __builtin_bit_cast(u32x4, vx);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] &= (zeros >> (2 * e) & 1 ? 0u : 0xffffu) | (zeros >> (2 * e + 1) & 1 ? 0u : 0xffff0000u);
            vx = __builtin_bit_cast(bf16x8, w);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
            acc[S][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(join_halves(fy[B][b][0], fy[B][b][1]), vx, acc[S][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    typedef std::integral_constant<int, 0> c0;
    typedef std::integral_constant<int, 1> c1;
    typedef std::integral_constant<int, 2> c2;

    if constexpr (MASKED) {  // rare: one stage, one step after the other
        for (int kt = 0; kt < nk; ++kt) {
            issue(0);
            wait_vmcnt<0>();
            barrier_nofence();
            read_y(c0{}, 0u);
            read_x(c0{}, 0u);
            read_x(c1{}, 0u);
            read_x(c2{}, 0u);
            lds_wait<0>(fx[2][1]);
            zeros = q_frag + 8 < (uint32_t)Qp ? 0u : column << ((uint32_t)Qp - 1 - q_frag);
            multiply(c0{}, c0{});
            multiply(c1{}, c0{});
            multiply(c2{}, c0{});
            q_frag = min(q_frag + q_step, q_frag + (q_step - (uint32_t)Qp));
            barrier_nofence();
        }
    } else {
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s) issue(s);
        wait_stages(std::integral_constant<int, STAGES - 2>{});
        barrier_nofence();
        read_y(c0{}, 0u);
        read_x(c0{}, 0u);
        read_x(c1{}, 0u);
        read_x(c2{}, 0u);
        constexpr int UNROLL = STAGES % 2 ? 2 * STAGES : STAGES;  // (the dy fragments alternate between two buffers)
        for (int kt0 = 0; kt0 < nk; kt0 += UNROLL) {
            static_for<0, UNROLL>([&](auto u_c) {
                constexpr int U = decltype(u_c)::value;
                if (kt0 + U < nk) {
                    wait_stages(std::integral_constant<int, STAGES - 3>{});  // the next stage has landed ...
                    barrier_nofence();  // ... for every wave, and nobody reads the previous one any more
                    typedef std::integral_constant<int, (U & 1)> now;
                    typedef std::integral_constant<int, ((U + 1) & 1)> next;
                    constexpr uint32_t nxt = (uint32_t)((U + 1) % STAGES) * kRow3StageBytes;
                    read_y(next{}, nxt);
                    multiply(c0{}, now{});
                    read_x(c0{}, nxt);
                    issue((U + STAGES - 1) % STAGES);
                    multiply(c1{}, now{});
                    read_x(c1{}, nxt);
                    multiply(c2{}, now{});
                    read_x(c2{}, nxt);
                }
            });
        }
    }
    lds_wait<0>(fx[0][0]);  // the fragments of the step past the end
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int s = 0; s < 3; ++s) lds_tie(fx[s][h]);
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int o = 0; o < 2; ++o) lds_tie(fy[b][o][h]);
    }
    wait_vmcnt<0>();  // the loads issued past the end have landed before LDS is reused

    // ---- the four position groups are added tap by tap, the middle one last: every wave parks its two blocks of 32 input x 32 output
    // channels, then wave w adds and stores half of block w >> 1 (rows and columns of an element as in wgrad_dl_body)
    float4* red = reinterpret_cast<float4*>(smem_b);
    int* again = reinterpret_cast<int*>(smem_b + kRow3ReduceBytes);  // one of each wave
    float probe = 0.f;
    int run_again = 0;
    const int row_pitch = a.direct ? a.RS * a.wpitch : a.out_row_pitch, tap_pitch = a.direct ? a.wpitch : a.CP;
    const int64_t first = (int64_t)n0 * row_pitch + (a.direct ? 0 : (int64_t)split * a.K * a.out_row_pitch);
    const uint32_t tile_bytes = (uint32_t)(min(a.K - n0, 64) * row_pitch) * 4u;
    const __amdgpu_buffer_rsrc_t o_srd = __builtin_amdgcn_make_buffer_rsrc(a.OUT + first, 0, tile_bytes, kBufFlags);
    const int blk = wave >> 1, g0 = (wave & 1) * 2;
    const int c = cb + (blk & 1) * 32 + (lane & 31), k0 = (blk >> 1) * 32 + 4 * (lane >> 5) + 8 * g0;
    const bool ok = c < (a.direct ? a.C : a.CP);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        constexpr int order[3] = {0, 2, 1};
        const int s = order[i];
        if (!MASKED && s == 1) {
            const bool any = __ballot(probe != probe && c < a.C) != 0;
            if (lane == 0) again[wave] = any;
        }
        __syncthreads();
        if (!MASKED && s == 1) {
#pragma unroll
            for (int w = 0; w < 8; ++w) run_again |= again[w];
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                red[((wp * 4 + b * 2 + wc) * 4 + g) * 64 + lane] =
                    make_float4(acc[s][b][4 * g], acc[s][b][4 * g + 1], acc[s][b][4 * g + 2], acc[s][b][4 * g + 3]);
        __syncthreads();
        float v[8];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            float4 r[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) r[w] = red[((w * 4 + blk) * 4 + g0 + g) * 64 + lane];
            v[4 * g] = ((r[0].x + r[1].x) + r[2].x) + r[3].x;
            v[4 * g + 1] = ((r[0].y + r[1].y) + r[2].y) + r[3].y;
            v[4 * g + 2] = ((r[0].z + r[1].z) + r[2].z) + r[3].z;
            v[4 * g + 3] = ((r[0].w + r[1].w) + r[2].w) + r[3].w;
        }
        if (!MASKED && s != 1) {  // (a sum is a NaN if one of its terms is; padding channels may hold anything)
            if (n0 + 64 <= a.K) {  // uniform
                probe += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) probe += n0 + k0 + 8 * (e >> 2) + (e & 3) < a.K ? v[e] : 0.f;
            }
        }
        const uint32_t at0 = ok ? (uint32_t)(k0 * row_pitch + (3 * fr + s) * tap_pitch + c) * 4u : kBufOut;
        auto at = [&](int e) { return at0 + (uint32_t)((8 * (e >> 2) + (e & 3)) * row_pitch) * 4u; };
        if (a.direct && a.lw) {  // uniform: regulariser folded in
            const __amdgpu_buffer_rsrc_t w_srd =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.lw) + first, 0, tile_bytes, kBufFlags);
            const float in = a.l_in && ok ? a.l_in[c] : 0.f;
            const float inv_in = in > 0.f ? 1.0f / in : 0.f;
            float wv[8], io[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                wv[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(w_srd, at(e), 0, 0));
                io[e] = a.l_on ? a.l_on[min(n0 + k0 + 8 * (e >> 2) + (e & 3), a.K - 1)] : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float inv_out = io[e] > 0.f ? 1.0f / io[e] : 0.f;
                v[e] += a.l_lambda * (wv[e] * (inv_out + inv_in));
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[e]), o_srd, at(e), 0, 0);
    }
    return __builtin_amdgcn_readfirstlane(run_again) != 0;
#else
    return false;
#endif
}

// One launch holds the weight gradients of up to kWgMaxProblems layers of any shape: every tile configuration and address
// mode is eight waves, so they are the branches of one kernel, and a workgroup finds its problem from the table of first
// workgroups (multiples of 8: workgroup ids are dealt round-robin to the 8 XCDs, and each XCD takes a contiguous range of
// every problem's split-major (split, tile) order - all tiles of one pixel split read the same x and dy slabs, which are
// then fetched into one L2 once).
constexpr int kWgMaxProblems = 20;
constexpr int kWgConfigs = 4;
struct WgradJobs {
    WgradArgs a[kWgMaxProblems];
    int first[64];
};
constexpr int kWgRow3 = kWgConfigs, kRow3Stages = 5;  // WgradArgs::cfg of wgrad_row3_body, which takes one layer a launch
// tile configurations (input channels x output channels) and pixels per reduction step
constexpr int kWgCfgBM[kWgConfigs] = {128, 64, 128, 64}, kWgCfgBN[kWgConfigs] = {128, 128, 64, 64};
constexpr int kWgCfgBKP[kWgConfigs] = {32, 64, 64, 64};
// LDS: five, four, four, five stages where fragments are read ahead, five, three, three, four where they are not
constexpr int kWgCfgLds[2][kWgConfigs] = {{80 * 1024, 72 * 1024, 72 * 1024, 64 * 1024}, {80 * 1024, 96 * 1024, 96 * 1024, 80 * 1024}};
// AHEAD: see the loop.  A launch that shares the chip with others does without it: their workgroups find room beside the
// smaller ring, and with other waves on the SIMD the latency is hidden anyway (training step of a pruned ResNet-50 -1.2 %).
template <int CFG, int XMODE, bool AHEAD>
__device__ __forceinline__ void wgrad_dl_cfg(const WgradArgs& a, int lin, uint8_t* smem) {
    constexpr int MORE = AHEAD ? 1 : 0;
    // 128 x 128: eight waves of 32 x 64 outputs, no wave groups; the others two groups of 2 x 2 waves
    if constexpr (CFG == 0) wgrad_dl_body<128, 128, 32, 4, 2, 5, 1, XMODE, AHEAD>(a, lin, smem);
    else if constexpr (CFG == 1) wgrad_dl_body<64, 128, 64, 2, 2, 3 + MORE, 2, XMODE, AHEAD>(a, lin, smem);
    else if constexpr (CFG == 2) wgrad_dl_body<128, 64, 64, 2, 2, 3 + MORE, 2, XMODE, AHEAD>(a, lin, smem);
    else wgrad_dl_body<64, 64, 64, 2, 2, 4 + MORE, 2, XMODE, AHEAD>(a, lin, smem);
}
template <int XMODE>
__device__ __forceinline__ void wgrad_dl_any(const WgradArgs& a, int lin, uint8_t* smem) {
    switch (a.cfg) {  // uniform
        case 0: wgrad_dl_cfg<0, XMODE, true>(a, lin, smem); break;
        case 1: wgrad_dl_cfg<1, XMODE, true>(a, lin, smem); break;
        case 2: wgrad_dl_cfg<2, XMODE, true>(a, lin, smem); break;
        default: wgrad_dl_cfg<3, XMODE, true>(a, lin, smem); break;
    }
}
__global__ __launch_bounds__(512, 1) void k_wgrad_dl_multi(const WgradJobs jobs) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_b[];
    const int ji = job_of_block(jobs.first, blockIdx.x);
    const WgradArgs a = jobs.a[ji];
    const int local = blockIdx.x - jobs.first[ji], n = a.tiles_m * a.tiles_n * a.splits;
    const int lin = (local & 7) * ((n + 7) >> 3) + (local >> 3);
    if (lin >= n) return;
    switch (a.xmode) {  // uniform
        case 0: wgrad_dl_any<0>(a, lin, smem_b); break;
        case 1: wgrad_dl_any<1>(a, lin, smem_b); break;
        default: wgrad_dl_any<2>(a, lin, smem_b); break;
    }
}
// One layer by itself: an instantiation of its own (its arguments one read of the kernel arguments away instead of two, no
// scalar registers spilled: 1 us of a call, 1.5 % of a training step that makes one call a layer).
template <int CFG, int XMODE, bool AHEAD>
__global__ __launch_bounds__(512, 1) void k_wgrad_dl(const WgradArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_b[];
    wgrad_dl_cfg<CFG, XMODE, AHEAD>(a, xcd_remap(blockIdx.x, gridDim.x), smem_b);
}
__global__ __launch_bounds__(512, 1) void k_wgrad_row3(const WgradArgs a) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_b[];
    const int lin = xcd_remap(blockIdx.x, gridDim.x);
    if (wgrad_row3_body<kRow3Stages, false>(a, lin, smem_b)) {
        __syncthreads();  // (everyone has seen that: the stage buffers are free)
        wgrad_row3_body<kRow3Stages, true>(a, lin, smem_b);
    }
}

// ------------------------------------------------------------------------------------------- //
// 3 x 3 convolution at stride 1, padding 1, with at most 64 channels on either side: weights resident in LDS
// ------------------------------------------------------------------------------------------- //
// The early 3 x 3 layers of a network (many pixels, few channels) have nine reduction steps per tile in the
// implicit-GEMM kernel, and a workgroup there spends as long on its set-up, its first loads and its stores as on the
// steps.  Here ONE workgroup per CU keeps the whole filter bank in LDS ([32 or 64 outputs][9 taps][16 * NCB channels] bf16,
// rows padded by 16 bytes, an odd number of 16-byte slots, so that the 32 rows a fragment read touches spread over all banks)
// and walks over a run of tiles of nby x nbx blocks of 4 x 8 output pixels (at most eight blocks, a patch of at most 348
// pixels: see r3_tile).  Per tile the input patch with its halo, (4*nby + 2) x (8*nbx + 2) pixels x 32, 64 or 128 bytes, goes
// to one of two LDS buffers by 16-byte global->LDS loads (out-of-image pixels and channels past the count fetch zeros), the
// next tile's patch while the current one is multiplied.  Wave b of the eight owns block b: 4 x 8 pixels x 64 outputs, two accumulator blocks; per
// (tap, 16 channels) one 16-byte patch read and two weight reads feed two MFMAs.  The nine taps are nine windows of the same patch: nothing is fetched twice.  The 16-byte
// chunks of a patch pixel are XOR-ed with ((column >> 1) & 3) | ((row & 1) << 2), and with as much of that as there are
// chunks to tell apart where a pixel has four or two: the 16 lanes one LDS cycle serves (two rows of eight pixels) then read
// 16 different bank groups, for every tap.  FLIP: the weights are indexed by the mirrored tap (input gradient: the same
// kernel on dy with the k-innermost filter copy).  The sums run over the filters' taps in their order, as in k_igemm_dl: the same bits.
//   A call of few tiles is bound by what comes ahead of its first MFMA: a load instruction costs a wave some 20 instructions
// of address and a CU's address unit 16 clocks, and one workgroup's worth of full-size bank and patch is 128 of them.  So bank
// and patch are laid out for the channels there are, and loads of filters past the last output (their rows only reach outputs
// that are not written) and past the end of a smaller patch are not made: 16 channels 80 -> 21 loads.  Against 64 channels'
// worth for every call, us: 128 x 32 x 32, 16 -> 16 5.97 -> 4.82, 16 x 16, 32 -> 32 4.65 -> 3.85, 8 x 8, 64 -> 64 5.40 -> 5.24,
// 16 x 16, 16 -> 16, batch 4 3.87 -> 2.95, 56 x 56, 64 -> 64, batch 64 23.2 -> 23.0; 54 layers forward 336 -> 299, input
// gradients 349 -> 309, none of them slower.  The test for the end of the patch stands in the set-up alone: in the tile loop,
// where its lanes are masked off anyway, it makes small patches 0.1 us faster and full ones 0.15 us slower.  More than one
// workgroup a CU, which the smaller LDS would allow, is up to 25 % slower: each loads the bank again.
struct Res3Args {
    const uint16_t* X;   // [N][H][W][ip]
    const uint16_t* Wt;  // [Mout][9][wp], reduction channel innermost
    uint16_t* Y;         // [N][H][W][op]
    int N, H, W, Cin, CinP, ip, Mout, wp, op;  // CinP = Cin rounded up to 8
    int nbx, nby;                            // blocks of 8 columns and of 4 rows per tile
    uint32_t pw_magic;                       // divides by the patch's width (fast_div)
    int tiles_x, tiles_y, tiles, run, patch_bytes;
    FastDiv x_div, y_div, bx_div;            // by tiles_x, tiles_y, nbx
    FastDiv cj_div;                          // by the 8-channel chunks of the output (KRSC)
};
constexpr int kR3TH = 4, kR3MaxNB = 7, kR3Waves = 8, kR3PatchPixels = (kR3TH + 2) * (8 * kR3MaxNB + 2);
constexpr int r3_rows(bool kb1) { return kb1 ? 64 : 32; }
constexpr int r3_wslots(int ncb) { return 18 * ncb + 1; }                                       // 16-byte slots per filter, the last one padding
constexpr int r3_wloads(int ncb, bool kb1) { return (r3_rows(kb1) * r3_wslots(ncb) + 63) / 64; }  // wave-level loads of 1 KB
constexpr int r3_chunks(int ncb) { return ncb == 1 ? 2 : ncb == 2 ? 4 : 8; }                    // 16-byte slots per patch pixel
constexpr int r3_ploads(int ncb) { return (kR3PatchPixels * r3_chunks(ncb) + 63) / 64; }
constexpr int r3_wbytes(int ncb, bool kb1) { return r3_wloads(ncb, kb1) * 1024; }
constexpr int r3_patch_bytes(int ncb, int pixels) { return pixels * r3_chunks(ncb) * 16; }
constexpr int kR3Slots = 256;  // one workgroup per CU
constexpr int kR3LdsMax = r3_wbytes(4, true) + 2 * r3_patch_bytes(4, kR3PatchPixels);
static_assert(kR3LdsMax <= 160 * 1024, "LDS plan");

// NCB: 16-channel steps per tap (CinP / 16 rounded up); KB1: more than 32 outputs (the second accumulator block is live).
// Compile-time so that the 9 * NCB steps of a tile are one straight line of code: with a branch per step every fragment
// read is waited out before its MFMA (27 us against 34 us for the implicit-GEMM kernel on 56 x 56 x 64 -> 64;
// straight-line with the reads of step s + 1 issued before the MFMAs of step s: see the numbers in the notes).
// KRSC (input gradient only): Wt is the layer's own filter bank [Cin = K][9][wp] with the output channel of this launch
// innermost, and the bank is transposed on its way into LDS: the loads of a workgroup's share all in flight, its 16-byte
// rows written as 2-byte elements.  A small layer is spared the launch that makes the k-innermost copy (16 x 16 channels,
// 16 x 16, batch 4: input gradient 2.6 + 2.9 us in two launches -> 3.2 us), but every workgroup transposes the whole bank and
// the 2-byte writes meet in the same LDS banks: up to 16 output channels it is 2 to 39 % faster for every K, beyond that 3 %
// slower to 33 % faster up to K * C = 768 (counted in eights), 11 % faster to 27 % slower (8 % in the middle) up to 1280, 2 %
// faster to 66 % slower (29 %) up to 2048, 24 to 124 % slower at 3072 (56 x 56, 33 -> 56 channels, batch 10: 10.1 us in two launches, 14.9 so).  Those take the two launches.
constexpr int kR3KrscFewC = 16, kR3KrscMaxBank = 768, kR3KrscBank = 64 * kR3KrscFewC;  // the largest that either rule takes
template <bool FLIP, int NCB, bool KB1, bool KRSC = false>
__global__ __launch_bounds__(512) void k_conv3x3_res(const Res3Args a) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr uint32_t kBufOut = 0xffffffffu, kBufFlags = 0x00020000u;
    constexpr int ROWS = r3_rows(KB1), WSLOTS = r3_wslots(NCB), WROW = WSLOTS * 16, WTAP = 32 * NCB;
    constexpr int NWL = r3_wloads(NCB, KB1), WL = (NWL + 7) / 8;  // wave-level loads of the weights, per wave
    constexpr int NCH = r3_chunks(NCB), NPL = r3_ploads(NCB), PL = (NPL + 7) / 8;
    constexpr int NKB = KB1 ? 2 : 1;  // accumulator blocks
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_b[];
    uint8_t* wl = smem_b;
    uint8_t* pbuf = smem_b + r3_wbytes(NCB, KB1);
    // where a patch pixel's 16-byte chunks lie (see above)
    auto chunk_xor = [](int pr, int pc) {
        return NCH == 2 ? pr & 1 : NCH == 4 ? ((pc >> 2) & 1) | ((pr & 1) << 1) : ((pc >> 1) & 3) | ((pr & 1) << 2);
    };
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int first = blockIdx.x * a.run, last = first + a.run < a.tiles ? first + a.run : a.tiles;
    if (first >= last) return;  // whole workgroup

    // ---- filter bank -> LDS, once ---------------------------------------------------------------------------------
    if constexpr (KRSC) {
        constexpr int IT = (kR3KrscBank / 8 * 9 + 511) / 512;  // 8 channels of one filter's tap an item
        const int ncj = (a.Mout + 7) >> 3, items = a.Cin * 9 * ncj;
        uint4 v[IT];
        int k9[IT], cj[IT];
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int it = min(tid + 512 * i, items - 1);
            k9[i] = (int)fdiv((uint32_t)it, a.cj_div);  // k * 9 + tap
            cj[i] = it - k9[i] * ncj;
            v[i] = *reinterpret_cast<const uint4*>(a.Wt + k9[i] * a.wp + cj[i] * 8);
        }
        // channels past the reduction's last one multiply zeros
        for (int sl = tid; sl < ROWS * WSLOTS; sl += 512) *reinterpret_cast<uint4*>(wl + sl * 16) = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            if (tid + 512 * i < items) {
                const int k = (int)__umulhi((uint32_t)k9[i], 0x1c71c71du), t = k9[i] - k * 9;  // (exact below 2^29)
                uint16_t* dst = reinterpret_cast<uint16_t*>(wl + cj[i] * 8 * WROW + t * WTAP + k * 2);
                const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
                for (int e = 0; e < 8; ++e) dst[e * (WROW / 2)] = (uint16_t)(w[e >> 1] >> ((e & 1) * 16));
            }
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): written before the first tile's barrier
    } else {
        const __amdgpu_buffer_rsrc_t w_srd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(a.Wt), 0, (uint32_t)(a.Mout * 9 * a.wp) * 2u, kBufFlags);
#pragma unroll
        for (int i = 0; i < WL; ++i) {
            const int idx = wave + 8 * i;  // uniform
            if (idx * 64 >= a.Mout * WSLOTS) break;  // (rows past the last output only reach outputs that are not written)
            const uint32_t sl = idx * 64 + lane, m = sl / WSLOTS, wi = sl - m * WSLOTS;  // (unsigned: no sign to correct for)
            const uint32_t t = wi / (2 * NCB), j = wi - t * (2 * NCB);
            const bool ok = wi < WSLOTS - 1 && (int)m < a.Mout && (int)(j * 8) < a.CinP;
            const uint32_t off = ok ? ((m * 9 + t) * a.wp + j * 8) * 2 : kBufOut;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w_srd, (lds_void_ptr)(wl + idx * 1024), 16, off, 0, 0, 0);
        }
    }
    // ---- this lane's slots of a patch: the same places in every tile ---------------------------------------------------
    const int pw = 8 * a.nbx + 2, patch_slots = (kR3TH * a.nby + 2) * pw * NCH;
    int p_rc[PL];        // row << 16 | column; -1: fetches zeros; -2: nothing there that is ever read
    uint32_t p_rel[PL];  // byte offset of the chunk from the patch's first pixel
    int p_idx[PL];
#pragma unroll
    for (int i = 0; i < PL; ++i) {
        p_idx[i] = wave + 8 * i;  // uniform
        p_rc[i] = -2, p_rel[i] = 0;
        if (p_idx[i] * 64 >= patch_slots) continue;
        const uint32_t sl = p_idx[i] * 64 + lane;
        const int pr = (int)fast_div(sl / NCH, a.pw_magic), pc = (int)(sl / NCH) - pr * pw, pj = (int)(sl % NCH);
        const int j = pj ^ chunk_xor(pr, pc);  // the logical chunk that belongs at this place
        p_rc[i] = (int)sl >= patch_slots || j >= 2 * NCB ? -2 : j * 8 < a.CinP ? (pr << 16) | pc : -1;
        p_rel[i] = (uint32_t)(((pr * a.W + pc) * a.ip + j * 8) * 2);
    }
    const uint32_t in_bytes = (uint32_t)(a.H * a.W * a.ip) * 2u, out_bytes = (uint32_t)(a.H * a.W * a.op) * 2u;
    auto decode = [&](int tile, int& tx, int& ty, int& img) {
        const int row = (int)fdiv((uint32_t)tile, a.x_div);
        img = (int)fdiv((uint32_t)row, a.y_div);
        tx = tile - row * a.tiles_x;
        ty = row - img * a.tiles_y;
    };
    auto issue = [&](int tile, int buf) {
        int tx, ty, img;
        decode(tile, tx, ty, img);
        const int ih0 = ty * kR3TH * a.nby - 1, iw0 = tx * 8 * a.nbx - 1;
        const __amdgpu_buffer_rsrc_t x_srd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(a.X) + (int64_t)img * a.H * a.W * a.ip, 0, in_bytes, kBufFlags);
        const uint32_t xs = (uint32_t)((ih0 * a.W + iw0) * a.ip * 2);
        uint8_t* dst = pbuf + buf * a.patch_bytes;
#pragma unroll
        for (int i = 0; i < PL; ++i) {
            const int ih = ih0 + (p_rc[i] >> 16), iw = iw0 + (p_rc[i] & 0xffff);
            const bool ok = p_rc[i] >= 0 && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            if (p_rc[i] != -2)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(x_srd, (lds_void_ptr)(dst + p_idx[i] * 1024), 16,
                                                         ok ? p_rel[i] + xs : kBufOut, 0, 0, 0);
        }
    };

    // ---- MFMA state -----------------------------------------------------------------------------------------------
    const int l32 = lane & 31, h = lane >> 5;
    const int by = (int)fdiv((uint32_t)wave, a.bx_div), bx = wave - by * a.nbx;
    const int pr0 = by * kR3TH + (l32 >> 3), pc0 = bx * 8 + (l32 & 7);  // this lane's output pixel inside the tile
    const bool active = by < a.nby;
    uint32_t pb[9], pk[9];  // per tap: byte offset of the pixel under it in a patch, and its chunk swizzle (<< 4)
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int pr = pr0 + t / 3, pc = pc0 + t % 3;
        pb[t] = (uint32_t)((pr * pw + pc) * (NCH * 16));
        pk[t] = (uint32_t)(chunk_xor(pr, pc) << 4);
    }
    const uint8_t* wa = wl + l32 * WROW + h * 16;
    const uint32_t hc = (uint32_t)(h << 4);

    issue(first, 0);
    int buf = 0;
    for (int tile = first; tile < last; ++tile, buf ^= 1) {
        const bool more = tile + 1 < last;  // uniform
        // the patch of this tile (and at first the weights) has landed; this wave's stores of the previous tile, which
        // were issued after those loads, may still be in flight (every active wave issues exactly 2 * NKB)
        if (active && tile != first) wait_vmcnt<2 * NKB>();
        else wait_vmcnt<0>();
        barrier_nofence();
        if (more) issue(tile + 1, buf ^ 1);
        // the loads stay here, ahead of the multiply and of the stores: the wait at the top of the next tile counts on
        // the stores being the last memory instructions of the wave, and the loads need the multiply's time to land
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if (active) {
            int tx, ty, img;
            decode(tile, tx, ty, img);
            f32x16 acc[NKB];
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[kb][v] = 0.f;
            const uint8_t* pp = pbuf + buf * a.patch_bytes;
            bf16x8 xb[2], w0[2], w1[2];
            auto read_frags = [&](auto s_c) {
                constexpr int S = decltype(s_c)::value, tw = S / NCB, cb = S % NCB, B = S & 1, t = FLIP ? 8 - tw : tw;
                xb[B] = *reinterpret_cast<const bf16x8*>(pp + pb[t] + (((uint32_t)(cb << 5) | hc) ^ pk[t]));
                w0[B] = *reinterpret_cast<const bf16x8*>(wa + tw * WTAP + cb * 32);
                if constexpr (KB1) w1[B] = *reinterpret_cast<const bf16x8*>(wa + 32 * WROW + tw * WTAP + cb * 32);
            };
            read_frags(std::integral_constant<int, 0>{});
            static_for<0, 9 * NCB>([&](auto s_c) {
                constexpr int S = decltype(s_c)::value, B = S & 1;
                if constexpr (S + 1 < 9 * NCB) read_frags(std::integral_constant<int, S + 1>{});
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w0[B], xb[B], acc[0], 0, 0, 0);
                if constexpr (KB1) acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[B], xb[B], acc[1], 0, 0, 0);
            });
            // ---- store: the lane-pair exchange of k_igemm_dl (64 contiguous bytes per pixel pair and output block) -----
            const __amdgpu_buffer_rsrc_t y_srd = __builtin_amdgcn_make_buffer_rsrc(
                a.Y + (int64_t)img * a.H * a.W * a.op, 0, out_bytes, kBufFlags);
            const int oh = ty * kR3TH * a.nby + pr0, ow = tx * 8 * a.nbx + pc0;
            const bool odd = (lane & 1) != 0;
            const int chl = (odd ? 16 : 0) + 8 * h;
            const bool row_ok = oh < a.H;
            const bool ok0 = row_ok && (ow & ~1) < a.W, ok1 = row_ok && (ow | 1) < a.W;
            const uint32_t pix0 = (uint32_t)((oh * a.W + (ow & ~1)) * a.op) * 2u;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                const int ch = kb * 32 + chl;
                const f32x16& c = acc[kb];
                uint32_t v[2][4];
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) {
                    const uint32_t x0 = cvt_pk_bf16(c[8 * gp + 0], c[8 * gp + 1]), y0 = cvt_pk_bf16(c[8 * gp + 2], c[8 * gp + 3]);
                    const uint32_t x1 = cvt_pk_bf16(c[8 * gp + 4], c[8 * gp + 5]), y1 = cvt_pk_bf16(c[8 * gp + 6], c[8 * gp + 7]);
                    const auto ps = __builtin_amdgcn_permlane32_swap(x0, x1, false, false);
                    const auto qs = __builtin_amdgcn_permlane32_swap(y0, y1, false, false);
                    v[gp][0] = ps[0]; v[gp][1] = qs[0]; v[gp][2] = ps[1]; v[gp][3] = qs[1];
                }
                uint32_t s0[4], s1[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t got = swap_lane_pair(odd ? v[0][e] : v[1][e]);
                    s0[e] = odd ? got : v[0][e];
                    s1[e] = odd ? v[1][e] : got;
                }
                uint4 o0 = make_uint4(s0[0], s0[1], s0[2], s0[3]), o1 = make_uint4(s1[0], s1[1], s1[2], s1[3]);
                const bool ch_ok = ch < a.Mout;
                if (ch_ok && ch + 7 >= a.Mout) {  // last chunk: zeros in its padding
                    const Mask8 k = make_mask8(a.Mout - ch);
                    o0 = mask8(o0, true, k);
                    o1 = mask8(o1, true, k);
                }
                const uint32_t off0 = pix0 + (uint32_t)ch * 2u;
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o0), y_srd, ok0 && ch_ok ? off0 : kBufOut, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o1), y_srd,
                                                       ok1 && ch_ok ? off0 + (uint32_t)a.op * 2u : kBufOut, 0, 0);
            }
        }
    }
#endif
}

// How many row blocks a tile has: the count that leaves the CU with the most tiles the fewest of them (an image of 32
// columns has four column blocks, i.e. work for four of the eight waves: with two row blocks the 32 x 32 layers of a
// CIFAR network at batch 128 are two tiles a CU instead of four), and of those the least, so that more CUs have one.
inline int64_t r3_tile(Res3Args& a) {
    const int nbw = (a.W + 7) / 8;
    a.nbx = nbw < kR3MaxNB ? nbw : kR3MaxNB;
    a.pw_magic = make_magic((uint32_t)(8 * a.nbx + 2));
    a.tiles_x = (a.W + 8 * a.nbx - 1) / (8 * a.nbx);
    const int64_t cols = (int64_t)a.N * a.tiles_x;
    int64_t best = INT64_MAX;
    for (int nby = 1; nby * a.nbx <= kR3Waves && (kR3TH * nby + 2) * (8 * a.nbx + 2) <= kR3PatchPixels; ++nby) {
        const int64_t run = (cols * ((a.H + kR3TH * nby - 1) / (kR3TH * nby)) + kR3Slots - 1) / kR3Slots;
        if (run < best) {
            best = run;
            a.nby = nby;
        }
    }
    a.tiles_y = (a.H + kR3TH * a.nby - 1) / (kR3TH * a.nby);
    return cols * a.tiles_y;
}

inline bool r3_krsc_bank_ok(int K, int C) { return C <= kR3KrscFewC || round_up(K, 8) * round_up(C, 8) <= kR3KrscMaxBank; }
enum Res3Kind { kRes3Fwd = 0, kRes3Bwd = 1, kRes3BwdKrsc = 2 };
inline hipError_t launch_conv3x3_res(Res3Args& a, Res3Kind kind, hipStream_t st) {
    const int ncb = (a.CinP + 15) / 16, kb1 = a.Mout > 32 ? 1 : 0;
    if (ncb < 1 || ncb > 4 || (kind == kRes3BwdKrsc && !r3_krsc_bank_ok(a.Cin, a.Mout))) return hipErrorInvalidValue;
    const int64_t tiles = r3_tile(a);
    if (tiles <= 0 || tiles > 0x3fffffff) return hipErrorInvalidValue;
    a.tiles = (int)tiles;
    a.run = (int)((tiles + kR3Slots - 1) / kR3Slots);
    a.x_div = make_fastdiv((int64_t)a.tiles_x);
    a.y_div = make_fastdiv((int64_t)a.tiles_y);
    a.bx_div = make_fastdiv((int64_t)a.nbx);
    a.cj_div = make_fastdiv((a.Mout + 7) / 8);
    const unsigned grid = (unsigned)((tiles + a.run - 1) / a.run);
    typedef void (*kern_t)(const Res3Args);
    static const kern_t kerns[3][4][2] = {
        {{k_conv3x3_res<false, 1, false>, k_conv3x3_res<false, 1, true>}, {k_conv3x3_res<false, 2, false>, k_conv3x3_res<false, 2, true>},
         {k_conv3x3_res<false, 3, false>, k_conv3x3_res<false, 3, true>}, {k_conv3x3_res<false, 4, false>, k_conv3x3_res<false, 4, true>}},
        {{k_conv3x3_res<true, 1, false>, k_conv3x3_res<true, 1, true>}, {k_conv3x3_res<true, 2, false>, k_conv3x3_res<true, 2, true>},
         {k_conv3x3_res<true, 3, false>, k_conv3x3_res<true, 3, true>}, {k_conv3x3_res<true, 4, false>, k_conv3x3_res<true, 4, true>}},
        // (more than 32 output and more than 16 reduction channels are a larger bank)
        {{k_conv3x3_res<true, 1, false, true>, k_conv3x3_res<true, 1, true, true>}, {k_conv3x3_res<true, 2, false, true>, nullptr},
         {k_conv3x3_res<true, 3, false, true>, nullptr}, {k_conv3x3_res<true, 4, false, true>, nullptr}}};
    static LdsOptIn opt_in[3][4][2];
    const kern_t kern = kerns[kind][ncb - 1][kb1];
    a.patch_bytes = r3_patch_bytes(ncb, (kR3TH * a.nby + 2) * (8 * a.nbx + 2));
    const int lds = r3_wbytes(ncb, kb1) + (a.run > 1 ? 2 : 1) * a.patch_bytes;
    if (hipError_t e = opt_in[kind][ncb - 1][kb1].ensure(reinterpret_cast<const void*>(kern), kR3LdsMax); e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(512), lds, st, a);
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------- //
// weight gradient of a network's first layer: image-like input, at most 4 channels at a pitch of 8
// ------------------------------------------------------------------------------------------- //
// dw[k][r][s][c] = sum over output pixels of dy[pixel][k] * x[pixel * stride + (r, s)][c] (Eq. 4).  As in k_stem_fwd
// the unit of work is a tile of output pixels (2 x 64) whose input patch is loaded once; here the dy tile comes along
// and both go to LDS by 16-byte global->LDS loads: dy rows of 64 channels = 128 bytes with the unit swizzle of
// k_wgrad_dl's 128-byte rows, the patch in image order at 16 bytes per pixel (the 4 padding channels ride along).
// The reduction runs over the tile's pixels, 16 per MFMA step: wave r of a group of eight owns filter row r and
// accumulates 64 output channels (two 32 x 32 blocks) x 32 columns = 8 taps x 4 channels.  Both fragments are
// transposing reads: of dy as in k_wgrad_dl; of the patch, a source lane points at the 4 channels of pixel
// (q + row) * stride + tap, so the 16 columns of a read are 4 taps x 4 channels and its rows 4 consecutive output
// pixels.  A workgroup has two such groups of eight waves working on alternate tiles of one run of tiles, each with
// its own double-buffered LDS region; at the end the second group's sums are added to the first's through LDS and ONE
// slab of fp32 partial sums per workgroup, [r][64][32], goes to the workspace.  One workgroup per CU: the slabs of a
// launch are 256 x 57 KB, summed in a fixed order by k_stem_wgrad_reduce (which also adds the regulariser's term).
struct StemWgradArgs {
    const uint16_t* X;   // [N][H][W][8]
    const uint16_t* DY;  // [N][P][Q][ypitch]
    float* PART;         // [workgroup][R][64][32]
    int N, H, W, P, Q, K, KP, R, S, pad_h, pad_w, ypitch;
    int tiles_q, tiles_p;  // tiles per image along Q and P
    int tiles, run;        // N * tiles_p * tiles_q, and how many consecutive tiles one workgroup takes
};
constexpr int kSwTH = 2, kSwTW = 64;
constexpr int kSwSlots = 256;                 // one workgroup of 16 waves per CU
constexpr int kSwPairsFrom = 17;              // tiles from which a workgroup takes at least two
constexpr int kSwSlabRow = 64 * 32;           // floats per filter row in a slab

template <int STRIDE>
__global__ __launch_bounds__(1024) void k_stem_wgrad(const StemWgradArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int PH = (kSwTH - 1) * STRIDE + kStemMaxR;   // patch rows (for the largest filter)
    constexpr int PW = (kSwTW - 1) * STRIDE + 8;           // patch columns: 8 taps per filter row
    constexpr int NXL = (PH * PW + 63) / 64;               // wave-level loads of a patch, 64 pixels each
    constexpr int XL = (NXL + 7) / 8;                      // per wave
    constexpr int YL = kSwTH * kSwTW / 8 / 8;              // dy: 8 pixels per wave-level load, 8 waves
    constexpr int YB = kSwTH * kSwTW * 128, XB = NXL * 1024, STAGE = YB + XB, GROUP = 2 * STAGE;
    constexpr uint32_t kBufOut = 0xffffffffu, kBufFlags = 0x00020000u;
    static_assert(YL == 2 && 2 * GROUP <= 160 * 1024, "tile config");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_b[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hh = wave >> 3, w8 = wave & 7;     // group of eight waves, wave inside it = filter row
    const int first = blockIdx.x * a.run, last = first + a.run < a.tiles ? first + a.run : a.tiles;
    const int niter = (a.run + 1) >> 1;          // the same for every workgroup: tiles past `last` are fetched as zeros
    const bool active = w8 < a.R;
    const int ph_used = (kSwTH - 1) * STRIDE + a.R;
    uint8_t* gbase = smem_b + hh * GROUP;

    // ---- loader state ---------------------------------------------------------------------------------------------
    // dy: wave-level load d = w8 + 8 i covers pixels 8 d .. 8 d + 7 of the tile (i = tile row), a lane one 16-byte chunk;
    // the chunk a lane fetches is the logical one that belongs at its physical place in the swizzled row
    const int yq = 8 * w8 + (lane >> 3);         // output column inside the tile
    uint32_t y_v[YL];
    {
        const int pc = lane & 7, sw = (yq >> 1) & 1;         // (the pixel row's swizzle bit: rows i * 64 + yq)
        const int qq = (pc >> 1) ^ sw;
        const int lc = ((((qq & 1) << 1) | (qq >> 1)) << 1) | (pc & 1);
#pragma unroll
        for (int i = 0; i < YL; ++i) y_v[i] = lc * 8 < a.KP ? (uint32_t)(((i * a.Q + yq) * a.ypitch + lc * 8) * 2) : kBufOut;
    }
    // patch: wave-level load idx covers pixels 64 idx .. 64 idx + 63 of the patch in row-major order; loads past the
    // last one repeat it (same data to the same place), so that every wave issues the same number
    int x_rc[XL];          // row << 16 | column, or -1
    uint32_t x_rel[XL];    // byte offset of the pixel from the patch's first pixel
    int x_idx[XL];
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        x_idx[i] = w8 + 8 * i < NXL ? w8 + 8 * i : NXL - 1;
        const int slot = x_idx[i] * 64 + lane;
        const int prow = slot / PW, pcol = slot - prow * PW;
        x_rc[i] = prow < ph_used && prow < PH ? (prow << 16) | pcol : -1;
        x_rel[i] = (uint32_t)(prow * a.W + pcol) * 16u;
    }
    const uint32_t img_bytes = (uint32_t)(a.H * a.W) * 16u;

    auto issue = [&](int tile, int stage) {
        const bool tv = tile < last;  // uniform
        const int tq = tile % a.tiles_q;
        const int tp = (tile / a.tiles_q) % a.tiles_p;
        const int img = tile / (a.tiles_q * a.tiles_p);
        const int p0 = tp * kSwTH, q0 = tq * kSwTW;
        uint8_t* sbase = gbase + stage * STAGE;
        const __amdgpu_buffer_rsrc_t y_srd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(a.DY) + ((int64_t)(img * a.P + p0) * a.Q + q0) * a.ypitch, 0, 0xffffff00u, kBufFlags);
        const bool q_ok = tv && q0 + yq < a.Q;
#pragma unroll
        for (int i = 0; i < YL; ++i) {
            const uint32_t v = q_ok && p0 + i < a.P ? y_v[i] : kBufOut;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(y_srd, (lds_void_ptr)(sbase + (w8 + 8 * i) * 1024), 16, v, 0, 0, 0);
        }
        const __amdgpu_buffer_rsrc_t x_srd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(a.X) + (int64_t)img * a.H * a.W * 8, 0, img_bytes, kBufFlags);
        const int ih0 = p0 * STRIDE - a.pad_h, iw0 = q0 * STRIDE - a.pad_w;
        const uint32_t xs = (uint32_t)((ih0 * a.W + iw0) * 16);
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const int ih = ih0 + (x_rc[i] >> 16), iw = iw0 + (x_rc[i] & 0xffff);
            const bool ok = tv && x_rc[i] >= 0 && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_srd, (lds_void_ptr)(sbase + YB + x_idx[i] * 1024), 16,
                                                     ok ? x_rel[i] + xs : kBufOut, 0, 0, 0);
        }
    };

    // ---- MFMA state -----------------------------------------------------------------------------------------------
    // transpose-read geometry: 16-lane group g16, lane t16; source lane t16 points at pixel row (t16 >> 2) and 8-byte
    // quad (t16 & 3); the result is 4 consecutive pixels for column 16 * (g16 & 1) + t16
    const int g16 = lane >> 4, t16 = lane & 15;
    const int tr_row = (g16 >> 1) * 8 + (t16 >> 2);   // + 4 h + 16 (step inside the tile row)
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_ptr)gbase;
    uint32_t ay[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int u = 2 * kb + (g16 & 1);              // 32-byte unit (16 channels) of the 128-byte row
        const int up = (((u & 1) << 1) | (u >> 1)) ^ ((tr_row >> 1) & 1);
        ay[kb] = lds0 + (uint32_t)(tr_row * 128 + (up << 5) + (t16 & 3) * 8);
    }
    // patch: filter row w8, pixel (tile column tr_row) * STRIDE + tap, tap = 4 (g16 & 1) + (t16 & 3)
    const uint32_t ax = lds0 + (uint32_t)(YB + (w8 * PW + tr_row * STRIDE + 4 * (g16 & 1) + (t16 & 3)) * 16);
    f32x16 acc[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[kb][v] = 0.f;

    // One tile: 8 steps of 16 pixels (tile row pl = step / 4); the reads of step st + 1 are in flight during the MFMAs of st.
    auto compute = [&](int stage) {
        const uint32_t sb = (uint32_t)(stage * STAGE);
        const uint32_t by0 = ay[0] + sb, by1 = ay[1] + sb, bx = ax + sb;
        s16x4 fy[2][2][2], fx[2][2];
        auto issue_reads = [&](auto st_c) {
            constexpr int ST = decltype(st_c)::value, PL = ST >> 2, KQ = ST & 3, B = ST & 1;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 0) {
                    fy[B][0][0] = lds_read_tr16_b64<(PL * 64 + 16 * KQ) * 128>(by0);
                    fy[B][1][0] = lds_read_tr16_b64<(PL * 64 + 16 * KQ) * 128>(by1);
                    fx[B][0] = lds_read_tr16_b64<(PL * STRIDE * PW + 16 * KQ * STRIDE) * 16>(bx);
                } else {
                    fy[B][0][1] = lds_read_tr16_b64<(PL * 64 + 16 * KQ + 4) * 128>(by0);
                    fy[B][1][1] = lds_read_tr16_b64<(PL * 64 + 16 * KQ + 4) * 128>(by1);
                    fx[B][1] = lds_read_tr16_b64<(PL * STRIDE * PW + (16 * KQ + 4) * STRIDE) * 16>(bx);
                }
            }
        };
        issue_reads(std::integral_constant<int, 0>{});
        static_for<0, 8>([&](auto st_c) {
            constexpr int ST = decltype(st_c)::value, B = ST & 1;
            if constexpr (ST + 1 < 8) {
                issue_reads(std::integral_constant<int, ST + 1>{});
                lds_wait<6>(fy[B][0][0]);
            } else {
                lds_wait<0>(fy[B][0][0]);
            }
            lds_tie(fy[B][0][1]); lds_tie(fy[B][1][0]); lds_tie(fy[B][1][1]); lds_tie(fx[B][0]); lds_tie(fx[B][1]);
            const bf16x8 vx = join_halves(fx[B][0], fx[B][1]);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(join_halves(fy[B][kb][0], fy[B][kb][1]), vx, acc[kb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // ---- tiles first + hh, first + hh + 2, ...: loads one tile ahead, one barrier per tile ------------------------------
    issue(first + hh, 0);
    for (int it = 0; it < niter; ++it) {
        wait_vmcnt<0>();      // this wave's loads of tile `it` have landed ...
        barrier_nofence();    // ... and everybody's; everybody is also done reading the other stage
        if (it + 1 < niter) issue(first + hh + 2 * (it + 1), (it + 1) & 1);
        if (active) compute(it & 1);
    }

    // ---- the second group's sums join the first's through LDS; one slab per workgroup ---------------------------------
    __syncthreads();
    float* red = reinterpret_cast<float*>(smem_b);
    if (hh == 1 && active) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) red[((w8 * 2 + kb) * 16 + v) * 64 + lane] = acc[kb][v];
    }
    __syncthreads();
    if (hh == 0 && active) {
        const int l32 = lane & 31, h = lane >> 5;
        float* slab = a.PART + ((int64_t)blockIdx.x * a.R + w8) * kSwSlabRow;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = kb * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                slab[k * 32 + l32] = acc[kb][v] + red[((w8 * 2 + kb) * 16 + v) * 64 + lane];
            }
    }
#endif
}

inline size_t stem_wgrad_lds(int stride) {
    const int ph = (kSwTH - 1) * stride + kStemMaxR, pw = (kSwTW - 1) * stride + 8;
    return (size_t)4 * (kSwTH * kSwTW * 128 + (ph * pw + 63) / 64 * 1024);
}

// Fills in the tiling; `slabs` = workgroups of the launch = slabs of partial sums written.
inline void plan_stem_wgrad(StemWgradArgs& a, int* slabs) {
    a.tiles_q = (a.Q + kSwTW - 1) / kSwTW;
    a.tiles_p = (a.P + kSwTH - 1) / kSwTH;
    const int64_t tiles = (int64_t)a.N * a.tiles_p * a.tiles_q;
    a.tiles = (int)tiles;
    // Tiles per workgroup: a pair (one for each wave group) takes 1.2 us, a slab 0.03 us to write and add up (fitted to 7 x 7
    // filters on 96 x 96 to 224 x 224 at batch 8 to 64: 192 tiles as 96 slabs 11 us, as 192 slabs 15 us).  The smallest
    // problems keep a tile and a slab for each workgroup, as pt_conv_bwd_weight_plan has always reported them: that is within
    // 0.2 us there (10 tiles 7.35 us, in pairs 7.16) and 1 us slower at 64 tiles.
    if (tiles < kSwPairsFrom) {
        a.run = 1;
        *slabs = (int)tiles;
        return;
    }
    const int64_t least = (tiles + kSwSlots - 1) / kSwSlots;
    float best = 1e30f;
    for (int64_t run = (least + 1) & ~1ll; run <= tiles + 1; run += 2) {
        const float tile_us = 0.6f * (float)run, us = tile_us + 0.03f * (float)((tiles + run - 1) / run);
        if (us < best) {
            best = us;
            a.run = (int)run;
        }
        if (tile_us > best) break;  // longer runs only get slower
    }
    *slabs = (int)((tiles + a.run - 1) / a.run);
}

inline hipError_t launch_stem_wgrad(const StemWgradArgs& a, int slabs, int stride, hipStream_t st) {
    const size_t lds = stem_wgrad_lds(stride);
    static LdsOptIn opt_in[2];
    if (stride == 1) {
        if (hipError_t e = opt_in[0].ensure(reinterpret_cast<const void*>(k_stem_wgrad<1>), lds); e != hipSuccess) return e;
        hipLaunchKernelGGL(k_stem_wgrad<1>, dim3((unsigned)slabs), dim3(1024), lds, st, a);
    } else {
        if (hipError_t e = opt_in[1].ensure(reinterpret_cast<const void*>(k_stem_wgrad<2>), lds); e != hipSuccess) return e;
        hipLaunchKernelGGL(k_stem_wgrad<2>, dim3((unsigned)slabs), dim3(1024), lds, st, a);
    }
    return hipSuccess;
}

}  // namespace pt
