// Conv2DBackpropFilter on gfx950 MFMA: Out[(kh,kw,ci)][co] = sum_p x-gather[p][(kh,kw,ci)] * dy[p][co],
// the reduction over p = (n, oh, ow) split across blockIdx.z and summed in split order.
#include "igemm_launch.h"

namespace tfk {

namespace {

struct BwfPlan {
    int bi, bj, splits, k_split;
    Igemm2Tile t;      // configuration of the pipelined kernel
};

BwfPlan bwf_plan_f32(const ConvShape &s);

// Tiles and split-K of one bwd-filter launch, chosen from sweeps over the AlexNet/VGG
// shapes: 128 x 128 tiles and the pixel reduction split into as many parts as keep the blocks
// within one full round of two blocks per CU (512 blocks): a last round with only a few blocks
// costs a whole block time, and more splits only add partial-sum traffic (AlexNet conv2-5:
// 357 us with four-block rounds, 297 us with this rule; the sustained two-stream AlexNet step
// 0.686 ms, against 0.694 with 384 blocks for the short launches).  64-channel layers, and
// multiples of 64 that are not of 128, take 64 x 128 tiles, layers of at most 32 output channels
// 32 x 128.  (192-channel tiles, which pay in the forward pass, need more registers here than two
// waves per SIMD have and spill.)
BwfPlan bwf_plan(int dt, const ConvShape &s, bool v2) {
    BwfPlan p;
    if (dt == 0 && v2) return bwf_plan_f32(s);
    const int bk = dt == 0 ? 32 : 64;
    const int m = s.KH * s.KW * s.C;
    // output channels a multiple of 64 but not of 128 (AlexNet conv2's 192): 64-channel tiles leave
    // none empty (128-channel ones would compute a quarter of the rows for nothing), and three of
    // their 48 KiB blocks fit a CU, so the splits fill one round of three (conv2: 95 -> 90 us)
    // Small products (up to 8 GFLOP over whole 64-channel tiles, 10 in 64 and more 128 x 128 tiles, of at most
    // 256): 64 x 64 tiles with three LDS stages; their splits reduce to fewer, shorter partials and their blocks overlap better
    // (14 x 14 x 512 -> 128, 1 x 1, batch 128: 17.0 -> 14.3 us; 28 x 28 x 192 -> 176, batch 128: 28.2 -> 21.5; over
    // random shapes up to 4 GFLOP 0.72-0.89 of the time, 4-8 0.75-0.92, 8-10 in fewer tiles 1.04, at most 1.45:
    // 7 x 95 x 95 x 112 -> 72, 3 x 3, 24.7 -> 35.8)
    // (with more tiles, or 128 over a few hundred pixels, there is no split and the output's bytes bound it:
    // 9216 -> 4096 over 128 rows 54 us with 64 x 64 tiles, 43 with 128 x 128; 126 x 7 x 3 x 800 -> 480, 3 x 3, 15.3
    // against 12.4; over fewer pixels the launch is short either way: 112 x 6 x 6 x 232 -> 160, 6 x 6, 4.6 against 6.3)
    const int64_t tiles128 = (int64_t)((s.K + 127) / 128) * ((m + 127) / 128);
    const double pixels = (double)s.N * s.OH * s.OW, flops = 2.0 * m * ((s.K + 63) / 64 * 64) * pixels;
    const bool small = v2 && s.K > 32 && tiles128 <= 256 && flops <= (tiles128 >= 64 ? 1e10 : 8e9) &&
                       (tiles128 < 128 || flops >= 1e9 || pixels < 256);
    const bool by64 = v2 && !small && s.K > 64 && s.K % 128 != 0 && s.K % 64 == 0;
    if (v2) {
        p.t = small ? Igemm2Tile{64, 64, 4, 3}
                    : (s.K > 64 && !by64 ? Igemm2Tile{128, 128, 4, 2}
                                         : (s.K > 32 ? Igemm2Tile{64, 128, 4, 2} : Igemm2Tile{32, 128, 4, 2}));
        p.bi = p.t.bi;
        p.bj = p.t.bj;
    } else {
        p.bi = igemm_bi(s.K);
        p.bj = 128;
    }
    const int tiles = ((s.K + p.bi - 1) / p.bi) * ((m + p.bj - 1) / p.bj);
    const int64_t ktot = (int64_t)s.N * s.OH * s.OW;
    const int64_t ktiles = (ktot + bk - 1) / bk;
    const int target = by64 ? 768 : 512;
    int64_t sp = target / tiles;
    const int64_t max_sp = std::max<int64_t>(1, ktiles / 8);   // at least 8 K tiles per split
    sp = std::max<int64_t>(1, std::min<int64_t>(sp, max_sp));
    sp = std::min<int64_t>(sp, 4096);
    const int64_t per = (ktiles + sp - 1) / sp;                 // K tiles per split
    p.k_split = (int)(per * bk);
    p.splits = (int)((ktiles + per - 1) / per);
    return p;
}

// fp32: 64 x 64 (32 x 64) tiles, splits that fill one round of three blocks per CU, and at most as
// many as the register-staged kernel's plan, whose partials size the workspace.
BwfPlan bwf_plan_f32(const ConvShape &s) {
    BwfPlan p;
    p.t = Igemm2Tile{igemm2_tiles_f32(s.K, 1 << 24, 1).bi, 64, 4, 3};
    p.bi = p.t.bi;
    p.bj = p.t.bj;
    const int tiles = ((s.K + p.bi - 1) / p.bi) * ((s.KH * s.KW * s.C + p.bj - 1) / p.bj);
    const int64_t ktiles = ((int64_t)s.N * s.OH * s.OW + 31) / 32;
    int64_t sp = std::min<int64_t>(std::max(1, 768 / tiles), bwf_plan(0, s, false).splits);
    const int64_t per = (ktiles + sp - 1) / sp;
    p.k_split = (int)(per * 32);
    p.splits = (int)((ktiles + per - 1) / per);
    return p;
}

size_t plan_ws(const ConvShape &s, const BwfPlan &p) {
    if (p.splits <= 1) return 0;
    return (size_t)p.splits * (size_t)s.KH * s.KW * s.C * s.K * sizeof(float);
}

}  // namespace

void conv_bwd_filter_plan(int dt, const ConvShape &s, int *splits, int *k_split) {
    const BwfPlan p = bwf_plan(dt, s, false);
    *splits = p.splits;
    *k_split = p.k_split;
}

size_t conv_bwd_filter_ws_bytes(int dt, const ConvShape &s) {
    size_t need = plan_ws(s, bwf_plan(dt, s, false));
    if (dt == 1) need = std::max(need, plan_ws(s, bwf_plan(dt, s, true)));
    if (conv_fold_applies(dt, s)) need = std::max(need, conv_fold_ws_bytes(2, s));
    if (dt == 1 && conv_band_bwf_applies(s, true))
        need = std::max(need, conv_band_x_bytes(s) + conv_band_bwf_partial_bytes(s, true));
    return need;
}

size_t conv_band_bwf_want_bytes(int dt, const ConvShape &s) {
    return dt == 1 && conv_band_bwf_applies(s, false) ? conv_band_x_bytes(s) + conv_band_bwf_partial_bytes(s, false) : 0;
}

template <typename T>
static hipError_t conv_bwd_filter_t(const void *x, int64_t xs, const void *dy, int64_t dys, float *dw,
                                    const ConvShape &s, void *ws, hipStream_t st) {
    constexpr int EPC = Elem<T>::kPerChunk;
    const int dti = sizeof(T) == 4 ? 0 : 1;
    IgArgs a;
    fill_geom(a, s);
    const int64_t mn = (int64_t)s.KH * s.KW * s.C * s.K;
    const int m = s.KH * s.KW * s.C;
    a.src_i = dy;
    a.src_j = x;
    a.xs = xs;
    a.ys = dys;
    a.NI = s.K;
    a.split_stride = mn;
    const bool vi = s.K % EPC == 0 && dys % EPC == 0 && aligned16p(dy);
    const bool vj = s.C % EPC == 0 && xs % EPC == 0 && aligned16p(x);
    hipError_t e;
    BwfPlan p;
    bool v2 = false;
    if (vi && vj && igemm2_fits(a, span_bytes((int64_t)s.N * s.OH * s.OW, dys, s.K, sizeof(T)),
                                span_bytes((int64_t)s.N * s.H * s.W, xs, s.C, sizeof(T)))) {
        p = bwf_plan(dti, s, true);
        v2 = p.splits > 1 || aligned16p(dw);
    }
    if (v2) {
        a.out = p.splits > 1 ? ws : (void *)dw;
        a.k_split = p.k_split;
        const bool done = sizeof(T) == 4 ? igemm2_launch_f32<DIR_BWD_FILTER>(a, m, p.splits, p.t, st)
                                         : igemm2_launch<DIR_BWD_FILTER>(a, m, p.splits, p.t, st);
        e = done ? hipGetLastError() : hipErrorInvalidValue;
    } else {
        p = bwf_plan(dti, s, false);
        a.out = p.splits > 1 ? ws : (void *)dw;
        a.k_split = p.k_split;
        e = igemm_launch<T, DIR_BWD_FILTER>(a, m, p.splits, vi, vj, st);
    }
    if (e != hipSuccess || p.splits <= 1) return e;
    return launch_sum_splits(reinterpret_cast<float *>(ws), p.splits, mn, dw, st);
}

hipError_t launch_conv_bwd_filter(int dt, const void *x, int64_t xs, const void *dy, int64_t dys, float *dw,
                                  const ConvShape &s, void *ws, size_t ws_bytes, hipStream_t st) {
    const size_t band = conv_band_bwf_want_bytes(dt, s);
    const bool base = band == 0 || ws_bytes < band;
    if (dt == 1 && conv_band_bwf_applies(s, base) && dys % 8 == 0 && aligned16p(dy) && aligned16p(ws)) {
        const int64_t npix = (int64_t)s.N * s.H * s.W;
        unsigned char *at = reinterpret_cast<unsigned char *>(ws);
        const bf16_t *x4 = rgbx_input(x, npix, s.C, xs, reinterpret_cast<bf16_t *>(at), st);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        float *part = reinterpret_cast<float *>(at + conv_band_x_bytes(s));
        return launch_conv_bwd_filter_band(x4, dy, dys, dw, s, part, base, st);
    }
    if (conv_fold_applies(dt, s) && dys % 8 == 0 && ((uintptr_t)dy & 15) == 0 && ((uintptr_t)ws & 15) == 0)
        return launch_conv_bwd_filter_folded(x, xs, dy, dys, dw, s, ws, st);
    if (conv_pad_applies(2, dt, s) && !conv_fold_applies(dt, s) && ws_bytes >= conv_pad_ws_bytes(2, dt, s)) {
        hipError_t e;
        if (conv_bwd_filter_padded(dt, x, xs, dy, dys, dw, s, ws, st, &e)) return e;
    }
    return dt == 0 ? conv_bwd_filter_t<float>(x, xs, dy, dys, dw, s, ws, st)
                   : conv_bwd_filter_t<bf16_t>(x, xs, dy, dys, dw, s, ws, st);
}

}  // namespace tfk
