// Host-side planning of the convolution launches: descriptor checks, kernel argument construction,
// tile-configuration choice and the split plan of the weight gradient.
#pragma once

#include <math.h>

#include "conv_kernels.h"

namespace pt {

inline int32_t check_desc(const pt_conv_desc* d) {
    if (!d) return PT_ERR_NULL;
    if (d->struct_size != sizeof(pt_conv_desc)) return PT_ERR_SHAPE;
    if (d->N <= 0 || d->H <= 0 || d->W <= 0 || d->C <= 0 || d->K <= 0 || d->R <= 0 || d->S <= 0) return PT_ERR_SHAPE;
    if (d->stride_h <= 0 || d->stride_w <= 0 || d->pad_h < 0 || d->pad_w < 0) return PT_ERR_SHAPE;
    if (d->H + 2 * d->pad_h < d->R || d->W + 2 * d->pad_w < d->S) return PT_ERR_SHAPE;
    if (d->P != (d->H + 2 * d->pad_h - d->R) / d->stride_h + 1) return PT_ERR_SHAPE;
    if (d->Q != (d->W + 2 * d->pad_w - d->S) / d->stride_w + 1) return PT_ERR_SHAPE;
    if (d->x_cpitch < d->C || d->y_cpitch < d->K || d->w_cpitch < d->C) return PT_ERR_SHAPE;
    if (d->flags & ~PT_CONV_PAD_ZERO) return PT_ERR_UNSUPPORTED;
    // limits of the 16/32-bit pixel arithmetic inside the kernels
    if (d->H > 16384 || d->W > 16384 || d->R > 255 || d->S > 255 || d->pad_h > 255 || d->pad_w > 255 ||
        d->stride_h > 255 || d->stride_w > 255)
        return PT_ERR_UNSUPPORTED;
    const int64_t in_pix = (int64_t)d->N * d->H * d->W, out_pix = (int64_t)d->N * d->P * d->Q;
    if (in_pix >= (1ll << 30) || out_pix >= (1ll << 30)) return PT_ERR_UNSUPPORTED;
    const int64_t big = d->H > d->W ? d->H : d->W;  // divisors of the in-kernel pixel decompositions
    if (in_pix * big >= (1ll << 32) || out_pix * big >= (1ll << 32)) return PT_ERR_UNSUPPORTED;
    // 32-bit element offsets into every tensor
    // (a margin below 2^31 elements: the buffer addressing of the direct kernels shifts offsets by up to a padded border)
    if (in_pix * d->x_cpitch >= (1ll << 31) - (1ll << 27) || out_pix * d->y_cpitch >= (1ll << 31) - (1ll << 27)) return PT_ERR_UNSUPPORTED;
    if ((int64_t)d->K * d->R * d->S * d->w_cpitch >= (1ll << 31)) return PT_ERR_UNSUPPORTED;
    if ((int64_t)d->C * d->R * d->S * round_up(d->K, 8) >= (1ll << 31)) return PT_ERR_UNSUPPORTED;
    if ((int64_t)d->R * d->S * round_up(d->C, 8) >= (1ll << 30)) return PT_ERR_UNSUPPORTED;
    if ((int64_t)d->R * d->S * round_up(d->K, 8) >= (1ll << 30)) return PT_ERR_UNSUPPORTED;
    return PT_OK;
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

inline IgemmArgs make_fwd_args(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, uint16_t* y) {
    IgemmArgs a{};
    a.A = x; a.B = w; a.D = y;
    a.pad_zero = (d->flags & PT_CONV_PAD_ZERO) != 0;
    a.zf_h = a.zf_w = 1;
    a.M = d->N * d->P * d->Q;
    a.gW = make_fastdiv((int64_t)d->Q); a.gH = make_fastdiv((int64_t)d->P);
    a.sW = make_smalldiv(d->Q); a.sH = make_smalldiv(d->P);
    a.srcH = d->H; a.srcW = d->W; a.apitch = d->x_cpitch;
    a.h_mul = d->stride_h; a.h_add = -d->pad_h; a.w_mul = d->stride_w; a.w_add = -d->pad_w;
    a.tr_step = 1; a.ts_step = 1; a.TR = d->R; a.TS = d->S;
    a.Cred = d->C; a.CredP = (int)round_up(d->C, 8);
    a.b_tap0 = 0; a.b_tr_stride = d->S; a.b_ts_stride = 1; a.b_taps = d->R * d->S;
    a.bpitch = d->w_cpitch; a.Nout = d->K;
    a.DH = d->P; a.DW = d->Q; a.d_hmul = 1; a.d_hadd = 0; a.d_wmul = 1; a.d_wadd = 0; a.dpitch = d->y_cpitch;
    a.d_linear = 1;
    a.fold = 0; a.TSm = d->S; a.Creal = d->C; a.Cfold = make_fastdiv((int64_t)a.CredP);
    a.d_vec = (d->y_cpitch % 4 == 0) && (((uintptr_t)y & 7) == 0);
    a.d_vec16 = (d->y_cpitch % 8 == 0) && aligned16(y);
    return a;
}

// One stride-parity class (ca, cb) of input pixels of the input-gradient problem: the pixels
// h = ca + stride_h*i, w = cb + stride_w*j, reached only by taps r = r0 + stride_h*jr, s = s0 + stride_w*js.
struct BwdClass {
    int gH, gW, r0, s0, TR, TS;
};

inline BwdClass bwd_data_class(const pt_conv_desc* d, int ca, int cb) {
    BwdClass c;
    c.gH = ca < d->H ? (d->H - ca + d->stride_h - 1) / d->stride_h : 0;
    c.gW = cb < d->W ? (d->W - cb + d->stride_w - 1) / d->stride_w : 0;
    c.r0 = (ca + d->pad_h) % d->stride_h;
    c.s0 = (cb + d->pad_w) % d->stride_w;
    c.TR = c.r0 < d->R ? (d->R - c.r0 + d->stride_h - 1) / d->stride_h : 0;
    c.TS = c.s0 < d->S ? (d->S - c.s0 + d->stride_w - 1) / d->stride_w : 0;
    return c;
}

inline IgemmArgs make_bwd_data_args(const pt_conv_desc* d, const BwdClass& c, int ca, int cb, const uint16_t* dy,
                                    const uint16_t* wt, uint16_t* dx) {
    const int kpitch = (int)round_up(d->K, 8);
    IgemmArgs a{};
    a.A = dy; a.B = wt; a.D = dx;
    a.pad_zero = (d->flags & PT_CONV_PAD_ZERO) != 0;  // the k-innermost weight copy always has zero padding
    a.zf_h = a.zf_w = 1;
    a.M = d->N * c.gH * c.gW;
    a.gW = make_fastdiv((int64_t)c.gW); a.gH = make_fastdiv((int64_t)c.gH);
    a.sW = make_smalldiv(c.gW); a.sH = make_smalldiv(c.gH);
    a.srcH = d->P; a.srcW = d->Q; a.apitch = d->y_cpitch;
    a.h_mul = 1; a.h_add = (ca + d->pad_h - c.r0) / d->stride_h;
    a.w_mul = 1; a.w_add = (cb + d->pad_w - c.s0) / d->stride_w;
    a.tr_step = -1; a.ts_step = -1; a.TR = c.TR; a.TS = c.TS;
    a.Cred = d->K; a.CredP = kpitch;
    a.b_tap0 = c.r0 * d->S + c.s0; a.b_tr_stride = d->stride_h * d->S; a.b_ts_stride = d->stride_w;
    a.b_taps = d->R * d->S; a.bpitch = kpitch; a.Nout = d->C;
    a.DH = d->H; a.DW = d->W; a.d_hmul = d->stride_h; a.d_hadd = ca; a.d_wmul = d->stride_w; a.d_wadd = cb;
    a.dpitch = d->x_cpitch;
    a.d_linear = (d->stride_h == 1 && d->stride_w == 1);
    a.fold = 0; a.TSm = c.TS; a.Creal = d->K; a.Cfold = make_fastdiv((int64_t)kpitch);
    a.d_vec = (d->x_cpitch % 4 == 0) && (((uintptr_t)dx & 7) == 0);
    a.d_vec16 = (d->x_cpitch % 8 == 0) && aligned16(dx);
    a.edge_prio = 1;
    return a;
}

// Small dense channel counts (an image-like input): fold the S taps of a filter row into one run (of at most the eight
// blocks that a table of tails has bytes for).
inline void igemm_fold(IgemmArgs& a) {
    if (a.fold || !(a.CredP < 64 && a.TS > 1 && a.ts_step == 1 && a.apitch == a.CredP && a.bpitch == a.CredP &&
                    a.b_ts_stride == 1 && a.TR * a.TS <= 64 && a.TS * a.CredP <= 512))
        return;
    a.fold = 1;
    a.TSm = a.TS;
    a.Creal = a.Cred;
    a.Cfold = make_fastdiv((int64_t)a.CredP);
    a.Cred = a.CredP = a.TS * a.CredP;
    a.TS = 1;
}

// Which kernel takes the problems of a call that fill less than one round of 128 x 128 tiles (`as`: one problem, or the
// stride-parity classes of an input gradient, which share a launch).  Estimated times in us: up to 256 workgroups take `steps`
// steps of t1 and f1 for set-up and stores, up to 512 (two on a CU, or one after the other) t2 and f2; z = what smaller tiles
// save of the stores of a 128 x 64 tile, as far as it is filled, where it also clears pixels that no tap reaches (zf_h * zf_w >
// 1).  Fitted to 3939 calls (random layers of 16 to 2048 channels at batch 1 to 128, layers of ResNet-50 at published and pruned
// widths), each in all forms, mean of operands in the caches and from memory: always one of them 38.61 / 37.07 / 41.63 ms,
// chosen 29.89, the best form of each call 29.80; 775 other calls 5.82 and 5.80.  What is fitted is a call's ratio to its best
// form: fitted to the sum of the times, in which calls of 3 us count for little, the choice took small tiles for reductions of
// one to four steps as well, where 128 x 64 tiles, with no partial tiles to add, are up to a quarter faster (1 x 1, 96 -> 32
// channels, 42 pixels: 3.38 -> 2.88 us), 314 of the calls more than 4 % above their best form; now 36.
// 0 = k_igemm_dl at 128 x 64, 1 = k_igemm_small at 64 x 64, 2 = at 32 x 32: all of them two workgroups on a CU.
inline int pick_igemm_kernel(const IgemmArgs* as, int n) {
    struct Est { int bm, bn, nb; float t1, t2, f1, f2, z; };
    constexpr int FORMS = 3;
    constexpr Est est[FORMS] = {{128, 64, 1, 0.373f, 0.423f, 0.346f, 2.114f, 0.f},
                                {64, 64, 1, 0.232f, 0.381f, 0.877f, 2.569f, 0.477f},
                                {32, 32, 2, 0.235f, 0.335f, 1.100f, 1.816f, 0.768f}};
    const bool clears = as[0].zf_h * as[0].zf_w > 1;  // (then it is the only class)
    const float filled = clears ? fminf((float)as[0].M, 128.f) * fminf((float)as[0].Nout, 64.f) / (128.f * 64.f) : 0.f;
    int best = 0;
    int64_t steps0 = 0;
    float best_us = 1e30f, us0 = 0.f;
    for (int k = 0; k < FORMS; ++k) {
        int64_t tiles = 0, tile_steps = 0, longest = 0;
        for (int i = 0; i < n; ++i) {
            const IgemmArgs& a = as[i];
            const int64_t t = ceil_div(a.M, est[k].bm) * ceil_div(a.Nout, est[k].bn);
            const int64_t steps = ceil_div(a.TR * a.TS * ceil_div(a.CredP, 64), est[k].nb);
            tiles += t;
            tile_steps += t * steps;
            longest = steps > longest ? steps : longest;
        }
        const int64_t full = tiles / 512, rem = tiles % 512;
        const float avg = (float)tile_steps / (float)tiles;
        const float last_steps = full ? avg : (float)longest;
        const float last = rem == 0 ? 0.f : rem <= 256 ? last_steps * est[k].t1 + est[k].f1 : last_steps * est[k].t2 + est[k].f2;
        const float us = (float)full * (avg * est[k].t2 + est[k].f2) + last - filled * est[k].z;
        if (k == 0) us0 = us, steps0 = longest;
        if (us < best_us) {
            best_us = us;
            best = k;
        }
    }
    // Up to five steps a near tie goes to 128 x 64 tiles: the call takes as long either way (82 such calls: within 1 % in the mean,
    // 6 % at most), but they reduce statistics in the same launch, and two problems of one call that choose the same share
    // theirs, where a second launch costs 3 us: 6 of 500 calls with statistics, 18 of 268 forward pairs and 10 of 268 pairs of
    // gradients of ResNet layers are up to 1.6 times as fast.
    return n == 1 && steps0 <= 5 && us0 <= best_us + 0.2f ? 0 : best;
}
constexpr int kIgemmLarge = 3;  // beyond pick_igemm_kernel's range: 128 x 128 tiles fill the chip
inline bool igemm_small_ok(const IgemmArgs& a) {  // no undefined channel padding, no statistics epilogue, a bit per tap
    return !a.stats && a.TR * a.TSm < 32 && ((a.fold ? a.Creal : a.Cred) % 8 == 0 || a.pad_zero);
}

// Which deep form of the direct kernel takes a problem, 0 = none: 1 = 128 x 128 and 2 = 256 x 128 in three stages.  `kernel` = what
// takes it otherwise.
// A call by itself: by estimated times (us).  The other forms, two workgroups on a CU: rounds of 512 tiles t2 a step and
// f2, a last one of up to 256 t1 and f1.  The deep forms hold a CU each (96 and 144 KB of LDS): rounds of 256 tiles.  Fitted to 820
// calls (random layers of at least 4 steps and 128 tiles of 128 x 64, batch 4 to 128, 65 to 2048 output channels), each in all
// forms with operands in the caches and from memory: without the deep forms 34.0 ms together, so 31.3, the best form for each
// 31.0; 7 of them more than 4 % slower than without, at most 1.09 times.  Layers of ResNet-50, batch 64, from memory: 14 x 14
// 1024 -> 256 16.6 -> 13.5 us, 3 x 3 256 -> 256 23.8 -> 20.3, 28 x 28 3 x 3 128 -> 128 20.3 -> 19.3.  128 x 64 tiles in six stages won
// nothing over them in three with the loads between the MFMAs (80 calls of 25 steps and more in one round: 5471 and 5426 us).
// Problems that share a launch stay with the other forms: two problems of one round each are two rounds here.
// Input gradients at stride 1 (the same loop; a strided one's classes share a launch) called by themselves as forward calls: 36
// layers of 4 to 128 images, 21 of them 1 to 36 % faster, the others the same: 14 x 14, 256 -> 256, 3 x 3 21.3 -> 17.6 us, 225 -> 207
// 23.1 -> 19.5, 1 x 1, 1024 -> 256 12.1 -> 10.4, 9 x 56 x 56, 517 -> 72, 3 x 3 53.2 -> 39.0.  In a batched call, also of one layer, they
// do without: beside weight gradients, which must find LDS beside them, the deep forms make the training step of ResNet-50 0.3 to 1 %
// longer.
inline int pick_igemm_deep(const IgemmArgs& a, int kernel, bool alone) {
    if (!alone || a.d_hmul * a.d_wmul > 1 || !igemm_small_ok(a) || a.fold || a.Nout <= 64) return 0;
    const int64_t nk = a.TR * a.TS * ceil_div(a.CredP, 64);
    const int64_t t128 = ceil_div(a.M, 128) * ceil_div(a.Nout, 128), t64 = ceil_div(a.M, 128) * ceil_div(a.Nout, 64);
    if (nk < 4 || t64 < 128 || (kernel != 0 && kernel != kIgemmLarge)) return 0;
    auto shared = [&](int64_t tiles, float t2, float f2, float t1, float f1) {
        const int64_t rem = tiles % 512, full = tiles / 512 + (rem > 256);
        return (float)full * ((float)nk * t2 + f2) + (rem > 0 && rem <= 256 ? (float)nk * t1 + f1 : 0.f);
    };
    auto own = [&](int64_t tiles, float t1, float f1) { return (float)ceil_div(tiles, 256) * ((float)nk * t1 + f1); };
    const float without = kernel == 0 ? shared(t64, 0.65f, 3.29f, 0.33f, 0.97f) : shared(t128, 0.77f, 4.21f, 0.90f, 1.05f);
    const float tall = own(ceil_div(a.M, 256) * ceil_div(a.Nout, 128), 0.66f, 5.26f), square = own(t128, 0.46f, 2.61f);
    if (fminf(tall, square) >= 0.98f * without) return 0;
    return square <= tall ? 1 : 2;
}

// Kernel and tile configuration.  `vec`: all operand rows are 16-byte aligned (pitches are multiples of 8
// elements) - then the direct global->LDS kernels are used, with a tall pixel tile for narrow outputs and small tiles
// where there are few.
// Unaligned pitches, and filters with more than 64 taps per launch (the direct kernel keeps one validity
// bit per tap in a 64-bit mask), take the register-staged kernel.
// `plan` == nullptr: the problem is launched.  Otherwise, when a direct kernel takes it, nothing is launched yet: the
// plan is filled in and *planned set, for launch_igemm_dl_planned to send it out together with other problems (the
// register-staged kernel is launched at once either way, *planned cleared).
// `kernel`: what pick_igemm_kernel said for the launch this problem will be part of, -1 = decide here.
// `alone`: the caller sends the planned problem out by itself.
inline hipError_t launch_igemm(IgemmArgs& a, bool vec, hipStream_t st, IgemmDlPlan* plan = nullptr, bool* planned = nullptr,
                               int kernel = -1, bool alone = false) {
    if (planned) *planned = false;
    if (!vec) return launch_igemm_cfg<128, 128, 32, 2, 2, 2, 2, false>(a, st);
    igemm_fold(a);
    if (a.TR * a.TSm > 64) return launch_igemm_cfg<128, 128, 32, 2, 2, 2, 2, true>(a, st);
    // 128x128 tiles when they still fill the chip, else 128x64 tiles (more workgroups, deeper pipeline)
    const int64_t tiles128 = ceil_div(a.M, 128) * ceil_div(a.Nout, 128);
    if (kernel < 0) kernel = tiles128 >= 256 ? kIgemmLarge : igemm_small_ok(a) ? pick_igemm_kernel(&a, 1) : 0;
    IgemmDlPlan own;
    IgemmDlPlan& p = plan ? *plan : own;
    const int deep = pick_igemm_deep(a, kernel, alone || plan == nullptr);
    hipError_t e;
    if (deep == 1) e = plan_igemm_dl_cfg<128, 128, 2, 4, 3, true>(a, p);
    else if (deep == 2) e = plan_igemm_dl_cfg<256, 128, 4, 2, 3, true>(a, p);
    else if (kernel == 2) e = plan_igemm_small_cfg<32, 32, 2, 4>(a, p);
    else if (kernel == 1) e = plan_igemm_small_cfg<64, 64, 1, 4>(a, p);
    // very many pixel tiles and a narrow output (the stem): tall tiles, so half as many workgroups pay set-up and fill
    else if (a.Nout <= 64 && tiles128 >= 4096 && !a.stats) e = plan_igemm_dl_cfg<256, 64, 4, 2, 2>(a, p);
    else if (a.Nout <= 64 || kernel != kIgemmLarge) e = plan_igemm_dl_cfg<128, 64, 4, 2, 3>(a, p);
    else e = plan_igemm_dl_cfg<128, 128, 2, 4, 2>(a, p);
    if (e != hipSuccess) return e;
    if (plan) {
        *planned = true;
        return hipSuccess;
    }
    return launch_igemm_dl_planned(&a, &p, 1, st);
}

inline size_t bwd_data_ws(const pt_conv_desc* d) {
    return (size_t)round_up((int64_t)d->C * d->R * d->S * round_up(d->K, 8) * 2, 256);
}

// Split plan of the weight gradient.  `dl`: the direct global->LDS kernel (one filter tap per tile row
// block, tiles of 64 or 128 channels) is used; otherwise the register-staged kernel (flattened
// (tap, channel) axis, fixed 128x128 tiles).
struct WgradPlan {
    int dl, fold, BM, BN, cfg;
    int bkp;  // output pixels per reduction step
    int splits, iters_total, iters_per_split, tiles_m, tiles_n, tiles_per_tap, CP, KP, Mtot;
    size_t ws_bytes;
};
constexpr int kWgBM = 128, kWgBN = 128, kWgBK = 32;  // register-staged kernel

// 64-wide tiles when 128-wide ones would waste more than ~20 % of their rows
inline int pick_tile(int n) {
    const int64_t r128 = round_up(n, 128), r64 = round_up(n, 64);
    return (r64 < r128 && r128 * 5 > (int64_t)n * 6) ? 64 : 128;
}

// What a reduction step and a split cost in a call with several layers, fitted to ResNet-50 layers on the chip (us): a step of
// the 128 x 128 tile takes 0.30 with one workgroup on the CU (smaller tiles: in proportion to their MFMAs, but no less than
// 0.6 of it), a split's tile of fp32 partial sums is written and read again at about 4 TB/s.
constexpr float kWgStepUs = 0.30f, kWgPartialUsPerByte = 2.f / 4e6f;
constexpr float kRow3Beside = 0.68f, kRow3Alone = 0.93f;
constexpr float kRow3StepUs = 0.28f;  // of wgrad_row3_body, 64 positions
constexpr int kWgMinSteps = 4;    // per workgroup
constexpr int kWgSlots = 256;     // one workgroup per CU: a second one on the CU finishes no more steps per microsecond
inline float wgrad_step_us(const WgradPlan& p) {
    if (p.cfg == kWgRow3) return kRow3StepUs;
    const float r = (float)p.BM * p.BN * p.bkp / (128.f * 128.f * 32.f);
    return kWgStepUs * (r > 0.6f ? r : 0.6f);
}

inline WgradPlan plan_wgrad_tiles(const pt_conv_desc* d, bool dl, int cfg = -1) {  // cfg: tile configuration, -1 = by the sizes
    // the direct kernel addresses the 128 rows of an output tile with 31 bits
    const int64_t row = (int64_t)d->R * d->S * (round_up(d->C, 8) > d->w_cpitch ? round_up(d->C, 8) : d->w_cpitch);
    dl = dl && row <= (1 << 22);
    WgradPlan p;
    p.dl = dl;
    p.CP = (int)round_up(d->C, 8);
    p.KP = (int)round_up(d->K, 8);
    p.Mtot = d->R * d->S * p.CP;
    p.cfg = 0;
    const int64_t pixels = (int64_t)d->N * d->P * d->Q;
    p.fold = dl && p.CP < 64 && d->S > 1 && d->x_cpitch == p.CP && d->w_cpitch == p.CP;
    if (dl) {
        const int run = p.fold ? d->S * p.CP : p.CP;  // contiguous elements of one tile row block
        p.BM = cfg >= 0 ? kWgCfgBM[cfg] : pick_tile(run);
        p.BN = cfg >= 0 ? kWgCfgBN[cfg] : pick_tile(p.KP);
        while (kWgCfgBM[p.cfg] != p.BM || kWgCfgBN[p.cfg] != p.BN) ++p.cfg;
        p.tiles_per_tap = (int)ceil_div(run, p.BM);
        p.tiles_m = (p.fold ? d->R : d->R * d->S) * p.tiles_per_tap;
        p.tiles_n = (int)ceil_div(d->K, p.BN);
        p.bkp = kWgCfgBKP[p.cfg];
    } else {
        p.bkp = kWgBK;
        p.BM = kWgBM;
        p.BN = kWgBN;
        p.tiles_per_tap = 0;
        p.tiles_m = (int)ceil_div(p.Mtot, kWgBM);
        p.tiles_n = (int)ceil_div(d->K, kWgBN);
    }
    p.iters_total = (int)ceil_div(pixels, p.bkp);
    return p;
}

// What wgrad_row3_body takes: 3 x 3 filters at stride 1 and padding 1 whose places and offsets fit its 24 and 30 bits (x is addressed
// from one pixel ahead of a slice, so the last channels of a single slice's last pixel end at (pixels + 1) * x_cpitch).
inline bool wgrad_row3_ok(const pt_conv_desc* d, bool dl) {
    const int64_t rows = (int64_t)d->N * d->H, pixels = rows * d->W, most = (int64_t)1 << 29;  // elements
    return dl && d->R == 3 && d->S == 3 && d->stride_h == 1 && d->stride_w == 1 && d->pad_h == 1 && d->pad_w == 1 &&
           pixels + rows < (1 << 24) && (pixels + 1) * d->x_cpitch <= most && pixels * d->y_cpitch < most;
}
inline WgradPlan plan_wgrad_row3(const pt_conv_desc* d, WgradPlan p) {  // p: the layer's plan in another form
    p.cfg = kWgRow3;
    p.fold = 0;
    p.BM = 3 * 64;
    p.BN = 64;
    p.bkp = kRow3Px;
    p.tiles_per_tap = (int)ceil_div(p.CP, 64);  // of one filter row
    p.tiles_m = 3 * p.tiles_per_tap;
    p.tiles_n = (int)ceil_div(d->K, 64);
    p.iters_total = (int)ceil_div((int64_t)d->N * d->H * (d->W + 1), kRow3Px);
    return p;
}
// One layer beside other kernels: the form whose workgroups spend less time on their steps together, the row form where that is
// well below (x 0.68: 256 -> 256 at 14 x 14 0.67, 64 -> 64 at 56 x 56 0.53; 512 -> 512 at 7 x 7, where an eighth of the positions
// are zeros, 0.71).  Times of workgroups: 14 x 14 72 of 53 us against 96 of 38, 56 x 56 153 of 52 against 96 of 36, 7 x 7 144 of 28
// against 192 of 26.  Step of ResNet-50, us in two runs, with the line at 0.60 (14 x 14 without), 0.68 and 0.75 (7 x 7 as well): batch 64 3270 and
// 3252, 3241 and 3228, 3242 and 3225; batch 48 2810 and 2800, 2795 and 2784, 2801 and 2803; batch 96 4545 and 4516, 4468 and 4504, 4537 and 4542;
// pruned 2713 and 2698, 2674 and 2702, 2674 and 2694; never 3273 and 3288, 2820 and 2827, 4556 and 4581, 2692 and 2723.  64, 80 and 128 workgroups a layer
// instead of 96: 0.4 to 0.8 % longer.  From 3000 pixels on: the row form's 2 us more of set-up and of adding up (5 x 13 x 13, 72 -> 40: 4.3
// us in 64 x 64 tiles, 7.1 so) are not in these times.  Steps at batch 8 and 12 are the same with the line and without
// (in five runs 0.4 % longer to 0.3 % shorter).
constexpr int64_t kRow3MinPixels = 3000;
inline WgradPlan plan_wgrad_beside(const pt_conv_desc* d, bool dl) {
    const WgradPlan p = plan_wgrad_tiles(d, dl);
    if (wgrad_row3_ok(d, p.dl) && (int64_t)d->N * d->P * d->Q >= kRow3MinPixels) {
        const WgradPlan r = plan_wgrad_row3(d, p);
        auto work = [](const WgradPlan& q) { return (float)q.tiles_m * q.tiles_n * q.iters_total * wgrad_step_us(q); };
        if (work(r) < kRow3Beside * work(p)) return r;
    }
    return p;
}

inline void set_wgrad_splits(const pt_conv_desc* d, WgradPlan& p, int64_t splits) {
    const int64_t most = p.iters_total / kWgMinSteps;
    if (splits > most) splits = most;
    if (splits < 1) splits = 1;
    p.iters_per_split = (int)ceil_div(p.iters_total, splits);
    p.splits = (int)ceil_div(p.iters_total, p.iters_per_split);
    p.ws_bytes = p.splits > 1 ? (size_t)round_up((int64_t)p.splits * d->K * p.Mtot * 4, 256) : 0;
}

// A call with one layer: tile configuration and splits that take the least time by what 672 shapes cost (ResNet layers,
// published and pruned, and random ones: 16 to 2048 channels, 5 to 56 pixels a side, batch 1 to 128), each in all
// configurations at 2 to 512 workgroups, with operands in the caches and with operands that come from memory, as in a
// training step; us: a step, a round of 256 workgroups (pipeline fill, stores), a megabyte of operands fetched into LDS by
// all workgroups together, a megabyte of partial sums written and read, the second launch.  Over all of them 128-wide tiles
// wherever they waste little take 12.05 ms (cached) and 14.41 ms (from memory), this choice 11.29 and 13.55, the best of
// each shape for both states together 11.15 and 13.22.  Costs fitted to cached operands alone: 11.31 and 13.73, by 64 x 128
// tiles with half the splits for large 1 x 1 layers, half as many operand bytes again (14 x 14 1024 -> 512 at batch 64: 23.4
// and 32.6 us against 23.3 and 26.5 so).
// The row form (wgrad_row3_body) where it is estimated at 0.93 of the others' best (mean of operands in the caches and from memory): of 102
// 3 x 3 layers of 3000 pixels and more the calls so chosen are within 0.3 % of the better form's in the mean (the line at 0.90 0.2 %, at 0.86
// 0.5 %, at 1.05 0.3 %), three up to 10 % slower than in the other form, most 5 to 34 % faster (21 x 39 x 40, 396 -> 192 89.5 -> 58.7 us); of 116
// smaller ones 0.2 % (0.90 0.4 %, 0.86 1.8 %, none at all some 10 %), five up to 9 % slower (1 x 47 x 50, 524 -> 359 19.2 and 21.0), others up to 40 %
// faster (4 x 22 x 22, 145 -> 1412 34.7 -> 20.6; 60 x 7 x 7, 512 -> 512 29.0 -> 26.3).
// Tiles smaller than the sizes ask for go unsplit up to 24 steps only (1536 pixels; 10 x 10 256 -> 256 3 x 3 at batch 15:
// 8.4 us against 12.5 split, from memory 10.3 and 14).  They are faster beyond that (14 x 14 at batch 8, 25 steps: 8.6 and
// 10.4 against 12.9 and 13.9): the line is not where measurements would put it.  The tests of the regulariser inside the
// wide reduction take layers of 1568 pixels, and ask pt_conv_bwd_weight_plan whether they are reduced so.
struct WgradCost {
    float step, round;
};
constexpr WgradCost kWgCost[kWgConfigs + 1] = {{0.257f, 1.343f}, {0.3f, 1.35f}, {0.312f, 1.388f}, {0.222f, 0.323f}, {0.32f, 6.5f}};
// The register-staged kernel on rows that are not 16-byte aligned (element-wise loads): 2.3 us a step.  Over 240 shapes at odd
// pitches its calls take 15.8 ms (cached) and 17.0 ms (from memory) so, with the 0.30 us of an aligned step 17.2 and 18.6.
constexpr WgradCost kWgStagedCost = {2.3f, 0.7f};
constexpr int kWgUnsplitSteps = 24;
constexpr float kWgPartialUsPerMB = 0.627f, kWgSecondUs = 1.065f, kWgOperandUsPerMB = 0.07f;
inline WgradPlan plan_wgrad(const pt_conv_desc* d, bool dl) {
    const WgradPlan own = plan_wgrad_tiles(d, dl);
    const bool direct = own.dl;
    WgradPlan best = own;
    const float part = (float)d->K * best.Mtot * 4e-6f * kWgPartialUsPerMB;  // of one split
    float best_us = 1e30f;
    const int forms = !direct ? 1 : wgrad_row3_ok(d, direct) ? kWgConfigs + 1 : kWgConfigs;
    for (int cfg = 0; cfg < forms; ++cfg) {
        const bool row3 = cfg == kWgRow3;  // (the last)
        if (row3) best_us *= kRow3Alone;
        const WgradPlan p = row3 ? plan_wgrad_row3(d, own) : plan_wgrad_tiles(d, dl, direct ? cfg : -1);
        const WgradCost cost = direct ? kWgCost[cfg] : kWgStagedCost;
        const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n, most = p.iters_total / kWgMinSteps;
        const float operands = (float)tiles * p.iters_total * p.bkp * ((row3 ? 64 : p.BM) + p.BN) * 2e-6f * kWgOperandUsPerMB;
        // none; around the optimum of steps / s + s * part without rounds; as many as fill one round or two
        const int64_t mid = (int64_t)fminf(sqrtf((float)p.iters_total * cost.step / part), 1e6f);
        const int64_t tries[7] = {1, mid - 1, mid, mid + 1, mid + mid / 4, kWgSlots / tiles, 2 * kWgSlots / tiles};
        for (int64_t s : tries) {
            if (s > most) s = most;
            if (s > 2 * kWgSlots / tiles) s = 2 * kWgSlots / tiles;
            if (s < 1) s = 1;
            WgradPlan q = p;
            set_wgrad_splits(d, q, s);
            if (q.splits == 1 && most > 1 && q.iters_total > kWgUnsplitSteps && direct && !row3 && (p.BM != own.BM || p.BN != own.BN)) continue;
            const float us = (float)ceil_div(q.splits * tiles, kWgSlots) * ((float)q.iters_per_split * cost.step + cost.round) +
                             (q.splits > 1 ? (float)q.splits * part + kWgSecondUs : 0.f) + operands;
            if (us < best_us) {
                best_us = us;
                best = q;
            }
        }
    }
    return best;
}

// The resident-weights kernel takes 3 x 3 filters at stride 1 and padding 1 with at most 64 channels on either side,
// 16-byte aligned rows, and channel counts that are multiples of 8 or the caller's PT_CONV_PAD_ZERO (the padding of the
// operand it reduces over must be zero, and it writes the output's last chunk whole, zeros in its padding).
// PT_RES3: bit 0 = forward calls, bit 1 = input-gradient calls, bit 2 = those of any filter bank size.
#ifndef PT_RES3
#define PT_RES3 3
#endif
constexpr int kRes3BwdMaxBank = 3072;  // K * C up to which an input gradient in a batched call takes the kernel
inline bool res3_shape_ok(const pt_conv_desc* d) {
    return d->R == 3 && d->S == 3 && d->stride_h == 1 && d->stride_w == 1 && d->pad_h == 1 && d->pad_w == 1 && d->C <= 64 &&
           d->K <= 64 && d->x_cpitch % 8 == 0 && d->y_cpitch % 8 == 0 &&
           (int64_t)d->H * d->W * (d->x_cpitch > d->y_cpitch ? d->x_cpitch : d->y_cpitch) * 2 <= 0x7fffffff;
}
// Larger banks (more than kRes3BwdMaxBank weights a tap) against the 128 x 64 tiles of k_igemm_dl, which add in the same order: by rounds of
// either, 256 of this kernel's tiles (a CU each) and 512 of those (two a CU; up to 256 of them are half a round).  us in those and
// here, from memory / cached, 64 -> 64 channels:
//   up to 256 tiles: 31 x 32 x 32 6.9 / 6.1 and 6.4 / 5.8, but beyond 32 columns, where a tile is one row of blocks, 33 columns 5.9 / 5.7 and
//   6.4 / 6.2 (batch 14), 10 x 56 x 56 6.8 / 5.9 and 7.4 / 6.6, 2 x 112 x 112 6.3 / 5.9 and 7.0 / 6.6;
//   up to 512, one round here (224 to 256 tiles): 18 x 56 x 56 9.9 / 8.2 and 8.9 / 7.2, 64 x 32 x 32 10.4 / 8.3 and 9.0 / 7.3, 64 x 28 x 28 9.6 /
//   7.9 and 8.5 / 7.1, with 168 of them 3 x 112 x 112 9.3 / 7.8 and 8.2 / 6.9; two rounds (280 to 400): 20 x 56 x 56 10.0 / 8.4 and 11.5 / 10.3, 80 x 28
//   x 28 10.2 / 8.4 and 11.5 / 10.4, 100 x 24 x 24 10.1 / 8.3 and 11.0 / 10.0, 40 x 40 x 40 10.1 / 8.3 and 11.4 / 10.1;
//   more, up to 0.8 of their tiles: 64 x 56 x 56 27.6 / 23.4 and 20.1 / 18.4, 64 x 48 x 48 21.0 / 18.0 and 16.8 / 14.7, 24 x 80 x 80 21.9 / 18.0 and
//   19.4 / 17.5, 100 x 40 x 40 22.1 / 18.1 and 18.3 / 17.1; more of them: 40 x 70 x 70 25.4 / 21.2 and 26.2 / 24.3, 128 x 33 x 33 20.3 / 17.7 and 20.2 / 19.4.
// 188 calls of both directions, mean of both states: always those tiles 1742 us, always these 1726, by this rule 1625, the better one of
// each 1624.  (From memory, calls of 500 tiles in k_igemm_dl took 15 to 18 us instead of 10 in one run of five, and two rounds here less.)
inline bool res3_large_ok(const pt_conv_desc* d) {
    const int64_t tiles = ceil_div((int64_t)d->N * d->H * d->W, 128);
    if (tiles <= 256) return d->W <= 32;
    Res3Args a{};
    a.N = d->N; a.H = d->H; a.W = d->W;
    const int64_t own = r3_tile(a);
    return tiles <= 512 ? own <= kR3Slots : 10 * own <= 9 * tiles;
}
inline bool res3_fwd_takes(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, const uint16_t* y) {
    return (PT_RES3 & 1) && res3_shape_ok(d) && d->w_cpitch % 8 == 0 && aligned16(x) && aligned16(w) && aligned16(y) &&
           ((d->C % 8 == 0 && d->K % 8 == 0) || (d->flags & PT_CONV_PAD_ZERO));
}
inline bool res3_fwd_ok(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, const uint16_t* y) {
    return res3_fwd_takes(d, x, w, y) && (d->C * d->K <= kRes3BwdMaxBank || res3_large_ok(d));
}
// launch_igemm's `kernel` of a forward call.  What the resident kernel takes and leaves to k_igemm_dl stays with its 128 x 64 tiles: they
// add in the same order, and with statistics (which the small tiles would leave to a second launch) y is the same and the call one
// launch.  us, small tiles / these / resident: 4 x 56 x 56, 64 -> 64 5.6, 5.8, 6.5 (with statistics 8.8, 6.9), 2 x 44 x 44, 64 -> 56 4.5, 5.3,
// 6.0 (8.0, 6.4), 8 x 36 x 36, 60 -> 64 5.5, 5.9, 6.2 (8.7, 7.2).
inline int fwd_kernel(const pt_conv_desc* d, const uint16_t* x, const uint16_t* w, const uint16_t* y) {
    return res3_fwd_takes(d, x, w, y) ? 0 : -1;
}
inline bool res3_bwd_ok(const pt_conv_desc* d, const uint16_t* dy, const uint16_t* wt, const uint16_t* dx, bool alone) {
    // (input-gradient launches share the chip with weight gradients on other streams, and a workgroup that holds a CU's
    // whole LDS for the length of the launch shuts those out: with the full 64 x 64 filter bank the train step gets
    // 25 us slower, with the smaller banks of a pruned network 25 us faster - so only those take it in batched calls)
    return (PT_RES3 & 2) && res3_shape_ok(d) && ((alone && res3_large_ok(d)) || PT_RES3 & 4 || d->C * d->K <= kRes3BwdMaxBank) && aligned16(dy) &&
           aligned16(wt) && aligned16(dx) &&
           ((d->C % 8 == 0 && d->K % 8 == 0) || (d->flags & PT_CONV_PAD_ZERO));
}

// The first layer's own weight-gradient kernel takes image-like inputs: at most 4 channels at a pitch of 8, at most 64
// output channels, a filter of at most 8 x 8 at stride 1 or 2, and sizes whose byte offsets fit its 32-bit addressing.
inline bool stem_wgrad_ok(const pt_conv_desc* d) {
    return d->C <= 4 && d->x_cpitch == 8 && d->y_cpitch % 8 == 0 && d->K <= 64 && d->stride_h == d->stride_w &&
           d->stride_h >= 1 && d->stride_h <= 2 && d->R <= kStemMaxR && d->S <= 8 &&
           (int64_t)d->H * d->W * 16 <= 0x7fffffff && ((int64_t)2 * d->Q + 64) * d->y_cpitch * 2 <= 0x7fffffff &&
           (int64_t)d->N * ((d->P + 1) / 2) * ((d->Q + 63) / 64) <= 0x3fffffff;
}

inline StemWgradArgs make_stem_wgrad_args(const pt_conv_desc* d, const uint16_t* x, const uint16_t* dy, float* part) {
    StemWgradArgs s{};
    s.X = x; s.DY = dy; s.PART = part;
    s.N = d->N; s.H = d->H; s.W = d->W; s.P = d->P; s.Q = d->Q; s.K = d->K; s.KP = (int)round_up(d->K, 8);
    s.R = d->R; s.S = d->S; s.pad_h = d->pad_h; s.pad_w = d->pad_w; s.ypitch = d->y_cpitch;
    return s;
}

// one slab of [R][64][32] floats per workgroup of the launch
inline size_t stem_wgrad_ws(const pt_conv_desc* d) {
    StemWgradArgs s = make_stem_wgrad_args(d, nullptr, nullptr, nullptr);
    int slabs = 0;
    plan_stem_wgrad(s, &slabs);
    return (size_t)round_up((int64_t)(slabs > 0 ? slabs : 1) * d->R * kSwSlabRow * 4, 256);
}

inline size_t wgrad_ws(const pt_conv_desc* d) {
    const size_t a = plan_wgrad(d, true).ws_bytes, b = plan_wgrad(d, false).ws_bytes;
    const size_t c = stem_wgrad_ok(d) ? stem_wgrad_ws(d) : 0;
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

// Workspace of the weight gradient with the regulariser folded into its reduction pass: at least one slab of partials
inline size_t wgrad_lasso_ws_of(const pt_conv_desc* d, const WgradPlan& p) {
    const size_t one = (size_t)round_up((int64_t)d->K * p.Mtot * 4, 256);
    return p.ws_bytes > one ? p.ws_bytes : one;
}

inline WgradArgs make_wgrad_args(const pt_conv_desc* d, const WgradPlan& p, const uint16_t* x, const uint16_t* dy,
                                 float* dw, void* ws) {
    WgradArgs a{};
    a.X = x; a.DY = dy;
    a.pixels = d->N * d->P * d->Q;
    a.Q = make_fastdiv((int64_t)d->Q); a.P = make_fastdiv((int64_t)d->P);
    a.sQ = make_smalldiv(d->Q); a.sP = make_smalldiv(d->P);
    a.H = d->H; a.W = d->W; a.xpitch = d->x_cpitch; a.ypitch = d->y_cpitch;
    a.stride_h = d->stride_h; a.stride_w = d->stride_w; a.pad_h = d->pad_h; a.pad_w = d->pad_w;
    a.S = d->S; a.RS = d->R * d->S; a.C = d->C; a.CP = p.CP; a.KP = p.KP; a.Mtot = p.Mtot; a.K = d->K;
    a.tiles_n = p.tiles_n; a.tiles_m = p.tiles_m; a.tiles_per_tap = p.tiles_per_tap; a.fold = p.fold;
    a.iters_total = p.iters_total; a.iters_per_split = p.iters_per_split; a.splits = p.splits;
    a.cfg = p.cfg;
    a.xmode = d->stride_h == 1 && d->stride_w == 1 && d->P == d->H && d->Q == d->W;
    if (a.xmode && d->R == 1 && d->S == 1 && d->pad_h == 0 && d->pad_w == 0) a.xmode = 2;
    a.dq = p.bkp % d->Q;
    a.dp = p.bkp / d->Q % d->P;
    a.dn = p.bkp / (d->P * d->Q);
    if (a.cfg == kWgRow3) {  // a place more in every row
        a.pixels = d->N * d->P * (d->Q + 1);
        a.Q = make_fastdiv((int64_t)d->Q + 1);
        a.dq = p.bkp % (d->Q + 1);
        a.dp = p.bkp / (d->Q + 1) % d->P;
    }
    a.wpitch = d->w_cpitch;
    a.direct = p.splits == 1;
    a.OUT = a.direct ? dw : (float*)ws;
    a.out_row_pitch = p.Mtot;
    a.o_vec = (d->w_cpitch % 4 == 0) && aligned16(dw);
    if (p.dl) {
        a.ntile_div = make_fastdiv((int64_t)p.tiles_m * p.tiles_n);
        a.tn_div = make_fastdiv(p.tiles_n);
        a.tap_div = make_fastdiv(p.tiles_per_tap);
        a.S_div = make_fastdiv((int64_t)d->S);
        a.CP_div = make_fastdiv((int64_t)p.CP);
    }
    return a;
}

// The direct kernel on one problem, or on a table of problems (then a multiple of 8 workgroups each, see
// k_wgrad_dl_multi).
template <int CFG, bool AHEAD>
inline hipError_t launch_wgrad_dl_one(const WgradArgs& a, hipStream_t st) {
    typedef void (*kern_t)(const WgradArgs);
    static const kern_t kerns[3] = {k_wgrad_dl<CFG, 0, AHEAD>, k_wgrad_dl<CFG, 1, AHEAD>, k_wgrad_dl<CFG, 2, AHEAD>};
    static LdsOptIn opt_in[3];
    constexpr size_t lds = (size_t)kWgCfgLds[AHEAD][CFG];
    if (hipError_t e = opt_in[a.xmode].ensure(reinterpret_cast<const void*>(kerns[a.xmode]), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(kerns[a.xmode], dim3((unsigned)(a.tiles_m * a.tiles_n * a.splits)), dim3(512), lds, st, a);
    return hipSuccess;
}
inline hipError_t launch_wgrad_row3(const WgradArgs& a, hipStream_t st) {
    constexpr size_t lds = (size_t)kRow3Stages * kRow3StageBytes;
    static LdsOptIn opt_in;
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void*>(k_wgrad_row3), lds); e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wgrad_row3, dim3((unsigned)(a.tiles_m * a.tiles_n * a.splits)), dim3(512), lds, st, a);
    return hipSuccess;
}
template <bool AHEAD>
inline hipError_t launch_wgrad_dl_cfg(const WgradArgs& a, hipStream_t st) {
    switch (a.cfg) {
        case 0: return launch_wgrad_dl_one<0, AHEAD>(a, st);
        case 1: return launch_wgrad_dl_one<1, AHEAD>(a, st);
        case 2: return launch_wgrad_dl_one<2, AHEAD>(a, st);
        case kWgRow3: return launch_wgrad_row3(a, st);
        default: return launch_wgrad_dl_one<3, AHEAD>(a, st);
    }
}
// beside: the launch shares the chip with others
inline hipError_t launch_wgrad_dl(WgradJobs& jobs, int n, bool beside, hipStream_t st) {
    if (n == 1) return beside ? launch_wgrad_dl_cfg<false>(jobs.a[0], st) : launch_wgrad_dl_cfg<true>(jobs.a[0], st);
    int64_t blocks = 0;
    int lds = 0;
    for (int i = 0; i < n; ++i) {
        if (kWgCfgLds[1][jobs.a[i].cfg] > lds) lds = kWgCfgLds[1][jobs.a[i].cfg];
        jobs.first[i] = (int)blocks;
        blocks += round_up((int64_t)jobs.a[i].tiles_m * jobs.a[i].tiles_n * jobs.a[i].splits, 8);
        if (blocks > 0x3fffffff) return hipErrorInvalidValue;
    }
    end_table(jobs.first, n);
    static LdsOptIn opt_in;
    if (hipError_t e = opt_in.ensure(reinterpret_cast<const void*>(k_wgrad_dl_multi), 160 * 1024); e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wgrad_dl_multi, dim3((unsigned)blocks), dim3(512), (size_t)lds, st, jobs);
    return hipSuccess;
}

}  // namespace pt
