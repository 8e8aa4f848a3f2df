// Conv2DBackpropInput on gfx950 MFMA, one stride phase per blockIdx.z:
// Out[p'][ci] = sum over the phase's taps (kh, kw) and co of dy[...][co] * w[kh][kw][ci][co].
#include "igemm_launch.h"

namespace tfk {

// The forward pass's tile rule.  (64 x 192 tiles for 33-64 input channels over many pixels copy
// 48 flop per byte against 64 x 128's 43 and ran AlexNet conv2's input gradient faster alone,
// 74.8 -> 71.3 us back to back, but the sustained two-stream step slower, 0.694 -> 0.705 ms, where
// the filter gradient of the other stream shares the GPU with it; GoogLeNet and Inception-v3
// steps are the same either way.)
static Igemm2Tile bwd_data_tiles(int dt, const ConvShape &s, int mj, int zdim) {
    return dt == 0 ? igemm2_tiles_f32(s.C, mj, zdim) : igemm2_tiles_narrow(s.C, mj, zdim, (int64_t)s.KH * s.KW * s.K);
}

// Tiles of the kernel fused with the ReLU backward, whose partial sums of the bias gradient (a row
// per block and wave column) go to the workspace: the rule's, where the workspace holds their
// rows (`all`), else without the tiles of fewer than 96 pixels (twice as many rows as 64 x 128).
static Igemm2Tile relu_tiles(int dt, const ConvShape &s, int mj, int zdim, bool all) {
    Igemm2Tile t = bwd_data_tiles(dt, s, mj, zdim);
    if (dt == 1 && !all && t.bj < 96) t = Igemm2Tile{64, 128, 4, 2};
    return t;
}

// Rows of bias-gradient partials of the fused ReLU-backward epilogue: one per block and wave
// column of the pipelined kernel's grid.
static int relu_partial_rows(int dt, const ConvShape &s, bool all) {
    const int mj = s.N * ((s.H + s.sh - 1) / s.sh) * ((s.W + s.sw - 1) / s.sw);
    const int z = s.sh * s.sw;
    const Igemm2Tile t = relu_tiles(dt, s, mj, z, all);
    return z * ((mj + t.bj - 1) / t.bj) * (t.nw / 2);
}

// Split-K at stride 1 (one phase) with few output tiles (fully connected layers and small late-
// stage images at small batch): fp32 partials in the workspace, then one epilogue pass (beta,
// or the fused ReLU backward with the bias-gradient rows after the partials).
static int bwd_data_splits(const ConvShape &s, int *k_split) {
    *k_split = 0;
    if (s.sh != 1 || s.sw != 1) return 1;
    return gemm_split_plan(s.C, s.N * s.H * s.W, (int64_t)s.KH * s.KW * s.K, k_split);
}

static size_t split_ws_bytes(int dt, const ConvShape &s, bool relu) {
    int ks;
    const int sp = bwd_data_splits(s, &ks);
    if (dt != 1 || sp <= 1) return 0;
    const int64_t mj = (int64_t)s.N * s.H * s.W;
    return (size_t)((sp + (relu ? 1 : 0)) * mj) * s.C * sizeof(float);
}

size_t conv_bwd_data_ws_bytes(int dt, const ConvShape &s) { return split_ws_bytes(dt, s, false); }

// ws: workspace (split-K partials; with relu_y also the bias-gradient partials).
// relu_y: the fused ReLU backward (of beta dx + the gradient); *db_parts / *db_at receive the number and place of
// the bias-gradient partial rows, or 0 when the fused kernels do not apply (nothing is launched
// then).
template <typename T>
static hipError_t conv_bwd_data_t(const void *dy, int64_t dys, const void *w, void *dx, int64_t dxs, float beta,
                                  const ConvShape &s, hipStream_t st, float *ws, const void *relu_y = nullptr,
                                  bool all = true, int *db_parts = nullptr, float **db_at = nullptr) {
    constexpr int EPC = Elem<T>::kPerChunk;
    IgArgs a;
    fill_geom(a, s);
    a.src_i = w;
    a.src_j = dy;
    a.out = dx;
    a.xs = dxs;
    a.ys = dys;
    a.beta = beta;
    a.NI = s.C;
    const bool vi = s.K % EPC == 0 && aligned16p(w);
    const bool vj = s.K % EPC == 0 && dys % EPC == 0 && aligned16p(dy);
    // largest phase: ceil(H / sh) x ceil(W / sw) pixels per image
    const int mj = s.N * ((s.H + s.sh - 1) / s.sh) * ((s.W + s.sw - 1) / s.sw);
    if constexpr (sizeof(T) == 2) {
        const int64_t wb = (int64_t)s.KH * s.KW * s.C * s.K * 2;
        if (vi && vj && s.C % 8 == 0 && dxs % 8 == 0 && aligned16p(dx) &&
            igemm2_fits(a, wb, span_bytes((int64_t)s.N * s.OH * s.OW, dys, s.K))) {
            const int z = s.sh * s.sw;
            int ks;
            const int sp = ws != nullptr && aligned16p(ws) ? bwd_data_splits(s, &ks) : 1;
            if (sp > 1) {
                a.k_split = ks;
                a.split_stride = (int64_t)mj * a.NI;
                a.out = ws;
                if (!igemm2_launch<DIR_BWD_DATA>(a, mj, sp, igemm2_tiles_split(a.NI, mj, sp, (int64_t)s.KH * s.KW * s.K), st))
                    return hipErrorInvalidValue;
                const hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
                SplitEpi ep{};
                ep.part = ws;
                ep.splits = sp;
                ep.rows = mj;
                ep.ni = a.NI;
                ep.split_stride = a.split_stride;
                ep.ostride = dxs;
                ep.out = dx;
                ep.beta = beta;
                ep.relu_y = relu_y;
                if (relu_y != nullptr) {                 // one partial row per output row
                    ep.db_part = ws + (int64_t)sp * mj * a.NI;
                    *db_parts = mj;
                    *db_at = ep.db_part;
                }
                return launch_split_epilogue(ep, st);
            }
            if (relu_y != nullptr) {
                a.relu_y = relu_y;
                a.db_part = ws;
                a.db_rows = relu_partial_rows(1, s, all);
                *db_parts = a.db_rows;
                *db_at = ws;
            }
            const Igemm2Tile t = relu_y != nullptr ? relu_tiles(1, s, mj, z, all) : bwd_data_tiles(1, s, mj, z);
            if (!igemm2_launch<DIR_BWD_DATA>(a, mj, z, t, st)) return hipErrorInvalidValue;
            return hipGetLastError();
        }
    }
    if constexpr (sizeof(T) == 4) {
        // (large tensors with short reductions, per stride phase on average, are bound by their stores, which the
        // register-staged kernel's wider tiles make in longer runs: 95 x 46 x 46 x 92 <- 12, 1 x 1, stride 2, 20.1
        // against 32.8 us.  With the ReLU backward the fused pass pays all the same.)
        const bool stores = relu_y == nullptr && (int64_t)s.KH * s.KW * s.K < 64 * s.sh * s.sw &&
                            (int64_t)s.N * s.H * s.W * s.C >= (4 << 20);
        if (!stores && vi && vj && s.C % EPC == 0 && dxs % EPC == 0 && aligned16p(dx) &&
            (relu_y == nullptr || aligned16p(relu_y)) &&
            igemm2_fits(a, (int64_t)s.KH * s.KW * s.C * s.K * 4, span_bytes((int64_t)s.N * s.OH * s.OW, dys, s.K, 4))) {
            if (relu_y != nullptr) {
                a.relu_y = relu_y;
                a.db_part = ws;
                a.db_rows = relu_partial_rows(0, s, true);
                *db_parts = a.db_rows;
                *db_at = ws;
            }
            if (!igemm2_launch_f32<DIR_BWD_DATA>(a, mj, s.sh * s.sw, bwd_data_tiles(0, s, mj, s.sh * s.sw), st))
                return hipErrorInvalidValue;
            return hipGetLastError();
        }
    }
    if (relu_y != nullptr) return hipSuccess;
    return igemm_launch<T, DIR_BWD_DATA>(a, mj, s.sh * s.sw, vi, vj, st);
}

size_t conv_bwd_data_relu_ws_bytes(int dt, const ConvShape &s, int64_t dxs) {
    int G;
    int64_t ppb;
    relu_bwd_plan(dt, (int64_t)s.N * s.H * s.W, s.C, dxs, &G, &ppb);
    const size_t fallback = (size_t)G * s.C * sizeof(float);
    if (dt != 1) return fallback;
    return std::max({fallback, (size_t)relu_partial_rows(1, s, false) * s.C * sizeof(float), split_ws_bytes(dt, s, true)});
}

// The rule's tiles (and fp32's fused kernel) may leave more partials than the workspace must hold:
// the query asks for room for them, and a call given less takes other tiles (fp32: the unfused pair).
size_t conv_bwd_data_relu_ws_want(int dt, const ConvShape &s, int64_t dxs) {
    return std::max({conv_bwd_data_relu_ws_bytes(dt, s, dxs), (size_t)relu_partial_rows(dt, s, true) * s.C * sizeof(float),
                     conv_pad_applies(3, dt, s) ? conv_pad_ws_bytes(3, dt, s) : 0});
}

hipError_t launch_conv_bwd_data_relu(int dt, const void *dy, int64_t dys, const void *w, void *dpre, int64_t dxs,
                                     const void *y, float beta, float *db, float *ws, size_t ws_bytes,
                                     const ConvShape &s, hipStream_t st, BiasPartials *defer) {
    if (conv_pad_applies(3, dt, s) && ws_bytes >= conv_pad_ws_bytes(3, dt, s)) {
        hipError_t e;
        BiasPartials bp{nullptr, 0};
        if (conv_bwd_data_padded(dt, dy, dys, w, dpre, dxs, beta, s, y, ws, st, &e, &bp)) {
            if (e != hipSuccess) return e;
            if (defer != nullptr) {
                *defer = bp;
                return hipSuccess;
            }
            return launch_sum_partials(bp.part, bp.rows, s.C, db, st);
        }
    }
    int parts = 0;
    float *db_at = nullptr;
    const bool all = ws_bytes >= conv_bwd_data_relu_ws_want(dt, s, dxs);
    if (dt == 1 ? ((uintptr_t)y & 7) == 0 : all) {
        const hipError_t e = dt == 1
            ? conv_bwd_data_t<bf16_t>(dy, dys, w, dpre, dxs, beta, s, st, ws, y, all, &parts, &db_at)
            : conv_bwd_data_t<float>(dy, dys, w, dpre, dxs, beta, s, st, ws, y, all, &parts, &db_at);
        if (e != hipSuccess) return e;
        if (parts > 0) {
            if (defer != nullptr) {
                defer->part = db_at;
                defer->rows = parts;
                return hipSuccess;
            }
            return launch_sum_partials(db_at, parts, s.C, db, st);
        }
    }
    // otherwise the two ops in sequence: the input gradient, then the ReLU backward in place
    const hipError_t e = launch_conv_bwd_data(dt, dy, dys, w, dpre, dxs, beta, s, nullptr, 0, st);
    if (e != hipSuccess) return e;
    return launch_bias_relu_bwd(dt, y, dpre, dpre, (int64_t)s.N * s.H * s.W, s.C, dxs, db, ws, st, defer);
}

hipError_t launch_conv_bwd_data(int dt, const void *dy, int64_t dys, const void *w, void *dx, int64_t dxs,
                                float beta, const ConvShape &s, float *ws, size_t ws_bytes, hipStream_t st) {
    if (conv_pad_applies(1, dt, s) && ws_bytes >= conv_pad_ws_bytes(1, dt, s)) {
        hipError_t e;
        if (conv_bwd_data_padded(dt, dy, dys, w, dx, dxs, beta, s, nullptr, ws, st, &e, nullptr)) return e;
    }
    return dt == 0 ? conv_bwd_data_t<float>(dy, dys, w, dx, dxs, beta, s, st, ws)
                   : conv_bwd_data_t<bf16_t>(dy, dys, w, dx, dxs, beta, s, st, ws);
}

}  // namespace tfk
