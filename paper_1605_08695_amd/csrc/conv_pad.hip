// Convolutions whose channel counts are not multiples of a 16-byte chunk (8 bf16 or 4 fp32 elements)
// on the pipelined implicit-GEMM kernels.
//
// Those kernels copy whole 16-byte chunks of one pixel's channels.  Other channel counts ran on the
// register-staged kernel, which gathers such operands one element at a time: 31 TFLOP/s for 108 x 29 x 29 x
// 1152 -> 74, 3 x 3, bf16.  Here the operands
// whose channel count is not a multiple are copied into the workspace with their channels padded with zeros
// (a pass over one activation and the filter), the product runs over the padded counts, and the output keeps
// its own layout: the forward and input-gradient epilogues store single elements (igemm2_kernel's RAG), and
// the filter gradient is summed into a padded filter and copied out.  The zeros add exact zeros to every
// sum.  It takes the workspace the query asks for; a call given less runs the register-staged kernel.
#include "igemm_launch.h"

namespace tfk {

namespace {

int chunk_of(int dt) { return dt == 0 ? 4 : 8; }
int up(int c, int e) { return (c + e - 1) / e * e; }
size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

ConvShape padded(int dt, const ConvShape &s) {
    ConvShape p = s;
    p.C = up(s.C, chunk_of(dt));
    p.K = up(s.K, chunk_of(dt));
    return p;
}

// Rows of C elements (stride xs) -> dense rows of Cp, zeros past C; one 16-byte chunk per thread.
template <typename T>
__global__ __launch_bounds__(256) void pad_rows_kernel(const T *__restrict__ x, int64_t chunks, int C, int64_t xs,
                                                       FastDiv dcpr, int cpr, T *__restrict__ xp) {
    constexpr int E = 16 / sizeof(T);
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < chunks; t += (int64_t)gridDim.x * 256) {
        int64_t row;
        int c;
        if (chunks < (1ll << 31)) {
            uint32_t q, r;
            dcpr.divmod((uint32_t)t, q, r);
            row = q;
            c = (int)r * E;
        } else {
            row = t / cpr;
            c = (int)(t - row * cpr) * E;
        }
        const T *src = x + row * xs + c;
        T v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = c + e < C ? src[e] : (T)0;
        *reinterpret_cast<U4 *>(xp + t * E) = *reinterpret_cast<const U4 *>(v);
    }
}

// w [taps][C][K] -> wp [taps][Cp][Kp], zeros past C and K; one 16-byte chunk per thread.
template <typename T>
__global__ __launch_bounds__(256) void pad_filter_kernel(const T *__restrict__ w, int taps, int C, int K, int Cp, int Kp,
                                                         T *__restrict__ wp) {
    constexpr int E = 16 / sizeof(T);
    const int64_t cpr = Kp / E, chunks = (int64_t)taps * Cp * cpr;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < chunks; t += (int64_t)gridDim.x * 256) {
        const int64_t row = t / cpr;
        const int k = (int)(t - row * cpr) * E;
        const int64_t tap = row / Cp;
        const int c = (int)(row - tap * Cp);
        const T *src = w + (tap * C + c) * K + k;
        T v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = c < C && k + e < K ? src[e] : (T)0;
        *reinterpret_cast<U4 *>(wp + t * E) = *reinterpret_cast<const U4 *>(v);
    }
}

// dwp [taps][Cp][Kp] -> dw [taps][C][K]
__global__ __launch_bounds__(256) void unpad_filter_kernel(const float *__restrict__ dwp, int64_t n, int C, int K, int Cp,
                                                           int Kp, float *__restrict__ dw) {
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < n; t += (int64_t)gridDim.x * 256) {
        const int64_t row = t / K, tap = row / C;
        dw[t] = dwp[(tap * Cp + (row - tap * C)) * Kp + (t - row * K)];
    }
}

unsigned grid_of(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 16384)); }

// x (pixel stride xs) itself when its chunks are whole and aligned, else a padded copy at *at
// (advanced past it).
template <typename T>
const void *pad_input(const void *x, int64_t pixels, int C, int Cp, int64_t &xs, unsigned char *&at, hipStream_t st) {
    constexpr int E = 16 / sizeof(T);
    if (C == Cp) return x;
    T *xp = reinterpret_cast<T *>(at);
    at += align256((size_t)pixels * Cp * sizeof(T));
    const int cpr = Cp / E;
    hipLaunchKernelGGL(pad_rows_kernel<T>, dim3(grid_of(pixels * cpr)), dim3(256), 0, st, (const T *)x, pixels * cpr, C, xs,
                       FastDiv((uint32_t)cpr), cpr, xp);
    xs = Cp;
    return xp;
}

template <typename T>
const void *pad_weights(const void *w, const ConvShape &s, const ConvShape &p, unsigned char *&at, hipStream_t st) {
    T *wp = reinterpret_cast<T *>(at);
    const int64_t n = (int64_t)s.KH * s.KW * p.C * p.K;
    at += align256((size_t)n * sizeof(T));
    hipLaunchKernelGGL(pad_filter_kernel<T>, dim3(grid_of(n * (int64_t)sizeof(T) / 16)), dim3(256), 0, st, (const T *)w,
                       s.KH * s.KW, s.C, s.K, p.C, p.K, wp);
    return wp;
}

size_t act_bytes(int dt, int64_t pixels, int C, int Cp) {
    return C == Cp ? 0 : align256((size_t)pixels * Cp * (dt == 0 ? 4 : 2));
}
size_t filter_bytes_padded(int dt, const ConvShape &p) {
    return align256((size_t)p.KH * p.KW * p.C * p.K * (dt == 0 ? 4 : 2));
}

// Input-gradient grid: largest stride phase and tile.
int phase_rows(const ConvShape &s) { return s.N * ((s.H + s.sh - 1) / s.sh) * ((s.W + s.sw - 1) / s.sw); }
Igemm2Tile bwd_tiles(int dt, const ConvShape &p) {
    const int64_t kred = (int64_t)p.KH * p.KW * p.K;
    return dt == 0 ? rag_tiles<float>(p.C, phase_rows(p), p.sh * p.sw, kred)
                   : rag_tiles<bf16_t>(p.C, phase_rows(p), p.sh * p.sw, kred);
}
int relu_rows(int dt, const ConvShape &p) {
    const Igemm2Tile t = bwd_tiles(dt, p);
    return p.sh * p.sw * ((phase_rows(p) + t.bj - 1) / t.bj) * (t.nw / 2);
}

}  // namespace

// From 1 MFLOP on, where the padded operands fit 32-bit byte offsets and nothing else handles the
// shape.  All directions of 14 x 14 x 30 -> 50, 3 x 3, batch 2 (11 MFLOP each): 178 -> 38 us, of
// 28 x 28 x 77 -> 50 (54 MFLOP) 301 -> 45, of 16 x 35 x 35 x 75 -> 100 (2.6 GFLOP) 381 -> 74; forward of
// 108 x 29 x 29 x 1152 -> 74, 3 x 3, stride 2: 1082 -> 146.
constexpr double kPadFlops = 1e6;

// The copies and the element-wise stores cost by the sizes of the tensors, the gather that they save by the
// reduction of each output, and in fp32 1 x 1 products by the arithmetic per element copied.  Random calls, padded
// against gathered:
//  * forward: fp32, and bf16 that copies x alone, below 64 elements 0.9-1.15 of the time (to 1.9; under 1M outputs
//    0.7-1), from there on 0.8 falling to 0.1; bf16 with ragged output channels gathers the filter too: 0.8 from
//    the shortest on.  fp32 1 x 1 that copies x, below 64 products per element: 0.95 under 8M elements, from there on
//    1.05-1.3, from 16M 1.1-1.45, from 32M 1.25-2.2 (3.1); larger filters 0.6-0.8, below 8 products from 32M 1.2;
//  * filter gradient: over few pixels there is little to gather, and the padded filter is copied out again: below 64
//    pixels 0.91-1.3 (to 1.9; 1M outputs and more 1.25-2.2, 128 pixels 1.1-1.5), then 0.85 falling to 0.3; bf16 with
//    ragged x 0.6-0.85 from 8 pixels on, over 2M outputs and more 1.07-1.35 below 64.  fp32 1 x 1 as in the forward
//    pass: 0.76-0.98 under 16M elements, 0.91-1.34 from there on, 1.09-2 from 32M;
//  * input gradient, by the largest stride phase's reduction: fp32 below 64 0.95-1.4 (to 2.5; under 1M outputs and
//    ragged dy 0.83-0.93 from 32 on), then 0.85 falling to 0.3; over 1M outputs it is the phases' average that
//    counts (the other phases only store): below 64 1.05-2.6; bf16 that copies dy under 1M outputs 0.75-0.87 from the
//    shortest on, over them below 64 0.87-1.8, then 0.98 falling to 0.2; bf16 whose dy is whole loses its vector
//    stores for nothing but the filter: 1-1.25 below 256, then 0.9 falling; over 1M outputs 1.15-2.2 below 512 on
//    average, then 0.8-1.15;
//  * fused with the ReLU backward it saves that pass: small tensors (4M elements) and bf16 with both counts ragged
//    gain from the shortest on, others from 64.
static bool pad_pays(int op, int dt, const ConvShape &s) {
    const bool ck = s.C % chunk_of(dt) != 0, kk = s.K % chunk_of(dt) != 0;
    const int64_t taps = (int64_t)s.KH * s.KW, px = (int64_t)s.N * s.H * s.W, py = (int64_t)s.N * s.OH * s.OW;
    if (op == 0 || op == 2) {
        const bool few = taps * s.K < (taps == 1 ? 64 : 8) * (int64_t)s.sh * s.sw;
        if (dt == 0 && ck && few && px * s.C >= (taps > 1 ? 32 : op == 0 ? 8 : 16) * (int64_t)(1 << 20)) return false;
    }
    if (op == 0) return (dt == 1 && kk) || taps * s.C >= 64 || py * s.K < (1 << 20);
    if (op == 2) {
        const int64_t out = taps * s.C * s.K;
        return py >= (dt == 1 && ck ? (out < (2 << 20) ? 8 : 64) : (out < (1 << 20) ? 64 : 128));
    }
    const int64_t red = taps * s.K / (s.sh * s.sw);
    if (op == 3) return (dt == 1 && ck && kk) || red >= 64 || px * s.C < (1 << 22);
    const int64_t most = (int64_t)((s.KH + s.sh - 1) / s.sh) * ((s.KW + s.sw - 1) / s.sw) * s.K;
    const bool big = px * s.C >= (1 << 20);
    if (dt == 0) return big ? red >= 64 : most >= (kk ? 32 : 64);
    return kk ? most >= 64 || !big : (big ? red >= 512 : most >= 256);
}

bool conv_pad_applies(int op, int dt, const ConvShape &s) {
    const int e = chunk_of(dt);
    const ConvShape p = padded(dt, s);
    if ((s.C % e == 0 && s.K % e == 0) || s.C < e || s.KH > 31 || s.KW > 31) return false;
    if (2.0 * s.N * s.OH * s.OW * s.KH * s.KW * (double)s.C * s.K < kPadFlops || !pad_pays(op, dt, s)) return false;
    constexpr int64_t kLim = int64_t(1) << 31;
    const int64_t es = 16 / e;
    return (int64_t)s.N * s.H * s.W * p.C * es < kLim && (int64_t)s.N * s.OH * s.OW * p.K * es < kLim &&
           (int64_t)s.KH * s.KW * p.C * p.K * 4 < kLim;
}

size_t conv_pad_ws_bytes(int op, int dt, const ConvShape &s) {
    const ConvShape p = padded(dt, s);
    const int64_t px = (int64_t)s.N * s.H * s.W, py = (int64_t)s.N * s.OH * s.OW;
    if (op == 0) return act_bytes(dt, px, s.C, p.C) + filter_bytes_padded(dt, p);
    if (op == 2)
        return act_bytes(dt, px, s.C, p.C) + act_bytes(dt, py, s.K, p.K) +
               align256((size_t)s.KH * s.KW * p.C * p.K * sizeof(float)) + align256(conv_bwd_filter_ws_bytes(dt, p));
    const size_t b = act_bytes(dt, py, s.K, p.K) + filter_bytes_padded(dt, p);
    return op == 1 ? b : b + align256((size_t)relu_rows(dt, p) * s.C * sizeof(float));
}

template <typename T>
static bool fwd_pad_t(int dt, const void *x, int64_t xs, const void *w, void *y, int64_t ys, const ConvShape &s,
                      const float *bias, void *ws, hipStream_t st, hipError_t *err) {
    const ConvShape p = padded(dt, s);
    if (s.C == p.C && (xs % (16 / (int)sizeof(T)) != 0 || !aligned16p(x))) return false;
    IgArgs a;
    fill_geom(a, p);
    // (an unpadded x keeps its pixel stride: its span must fit 32-bit offsets too)
    const int64_t px = (int64_t)s.N * s.H * s.W;
    if (!igemm2_fits(a, (int64_t)p.KH * p.KW * p.C * p.K * sizeof(T),
                     span_bytes(px, s.C == p.C ? xs : p.C, p.C, sizeof(T)))) return false;
    unsigned char *at = reinterpret_cast<unsigned char *>(ws);
    a.src_j = pad_input<T>(x, px, s.C, p.C, xs, at, st);
    a.src_i = pad_weights<T>(w, s, p, at, st);
    a.out = y;
    a.xs = xs;
    a.ys = ys;
    a.NI = p.K;
    a.ni_store = s.K;
    a.bias = bias;
    const int mj = s.N * s.OH * s.OW;
    *err = igemm2_launch_rag<T, DIR_FWD>(a, mj, 1, rag_tiles<T>(a.NI, mj, 1, (int64_t)p.KH * p.KW * p.C), st);
    return true;
}

template <typename T>
static bool bwd_data_pad_t(int dt, const void *dy, int64_t dys, const void *w, void *dx, int64_t dxs, float beta,
                           const ConvShape &s, const void *relu_y, void *ws, hipStream_t st, hipError_t *err,
                           BiasPartials *parts) {
    const ConvShape p = padded(dt, s);
    if (s.K == p.K && (dys % (16 / (int)sizeof(T)) != 0 || !aligned16p(dy))) return false;
    IgArgs a;
    fill_geom(a, p);
    const int64_t py = (int64_t)s.N * s.OH * s.OW;
    if (!igemm2_fits(a, (int64_t)p.KH * p.KW * p.C * p.K * sizeof(T),
                     span_bytes(py, s.K == p.K ? dys : p.K, p.K, sizeof(T)))) return false;
    unsigned char *at = reinterpret_cast<unsigned char *>(ws);
    if (relu_y != nullptr) {
        a.relu_y = relu_y;
        a.db_part = reinterpret_cast<float *>(at);
        a.db_rows = relu_rows(dt, p);
        at += align256((size_t)a.db_rows * s.C * sizeof(float));
        parts->part = a.db_part;
        parts->rows = a.db_rows;
    }
    a.src_j = pad_input<T>(dy, py, s.K, p.K, dys, at, st);
    a.src_i = pad_weights<T>(w, s, p, at, st);
    a.out = dx;
    a.xs = dxs;
    a.ys = dys;
    a.NI = p.C;
    a.ni_store = s.C;
    a.beta = beta;
    *err = igemm2_launch_rag<T, DIR_BWD_DATA>(a, phase_rows(p), s.sh * s.sw, bwd_tiles(dt, p), st);
    return true;
}

template <typename T>
static bool bwd_filter_pad_t(int dt, const void *x, int64_t xs, const void *dy, int64_t dys, float *dw, const ConvShape &s,
                             void *ws, hipStream_t st, hipError_t *err) {
    constexpr int E = 16 / sizeof(T);
    const ConvShape p = padded(dt, s);
    if ((s.C == p.C && (xs % E != 0 || !aligned16p(x))) || (s.K == p.K && (dys % E != 0 || !aligned16p(dy)))) return false;
    unsigned char *at = reinterpret_cast<unsigned char *>(ws);
    const void *xp = pad_input<T>(x, (int64_t)s.N * s.H * s.W, s.C, p.C, xs, at, st);
    const void *dyp = pad_input<T>(dy, (int64_t)s.N * s.OH * s.OW, s.K, p.K, dys, at, st);
    float *dwp = reinterpret_cast<float *>(at);
    at += align256((size_t)s.KH * s.KW * p.C * p.K * sizeof(float));
    *err = launch_conv_bwd_filter(dt, xp, xs, dyp, dys, dwp, p, at, 0, st);
    if (*err != hipSuccess) return true;
    const int64_t n = (int64_t)s.KH * s.KW * s.C * s.K;
    hipLaunchKernelGGL(unpad_filter_kernel, dim3(grid_of(n)), dim3(256), 0, st, dwp, n, s.C, s.K, p.C, p.K, dw);
    *err = hipGetLastError();
    return true;
}

bool conv_fwd_padded(int dt, const void *x, int64_t xs, const void *w, void *y, int64_t ys, const ConvShape &s,
                     const float *bias, void *ws, hipStream_t st, hipError_t *err) {
    return dt == 0 ? fwd_pad_t<float>(dt, x, xs, w, y, ys, s, bias, ws, st, err)
                   : fwd_pad_t<bf16_t>(dt, x, xs, w, y, ys, s, bias, ws, st, err);
}

bool conv_bwd_data_padded(int dt, const void *dy, int64_t dys, const void *w, void *dx, int64_t dxs, float beta,
                          const ConvShape &s, const void *relu_y, void *ws, hipStream_t st, hipError_t *err,
                          BiasPartials *parts) {
    return dt == 0 ? bwd_data_pad_t<float>(dt, dy, dys, w, dx, dxs, beta, s, relu_y, ws, st, err, parts)
                   : bwd_data_pad_t<bf16_t>(dt, dy, dys, w, dx, dxs, beta, s, relu_y, ws, st, err, parts);
}

bool conv_bwd_filter_padded(int dt, const void *x, int64_t xs, const void *dy, int64_t dys, float *dw, const ConvShape &s,
                            void *ws, hipStream_t st, hipError_t *err) {
    return dt == 0 ? bwd_filter_pad_t<float>(dt, x, xs, dy, dys, dw, s, ws, st, err)
                   : bwd_filter_pad_t<bf16_t>(dt, x, xs, dy, dys, dw, s, ws, st, err);
}

}  // namespace tfk
