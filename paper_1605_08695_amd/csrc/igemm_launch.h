// Host-side launch of the implicit-GEMM kernel: tile choice, vector-path
// selection and grid shape.
#pragma once
#include <utility>

#include "igemm.h"
#include "igemm2.h"
#include "kernels.h"

namespace tfk {

static inline bool aligned16p(const void *p) { return ((uintptr_t)p & 15) == 0; }

template <typename T, int DIR, int BI>
static void igemm_dispatch(const IgArgs &a, dim3 grid, bool vi, bool vj, hipStream_t st) {
    if (vi && vj)
        hipLaunchKernelGGL((igemm_kernel<T, DIR, BI, 128, true, true>), grid, dim3(256), 0, st, a);
    else if (vi)
        hipLaunchKernelGGL((igemm_kernel<T, DIR, BI, 128, true, false>), grid, dim3(256), 0, st, a);
    else if (vj)
        hipLaunchKernelGGL((igemm_kernel<T, DIR, BI, 128, false, true>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((igemm_kernel<T, DIR, BI, 128, false, false>), grid, dim3(256), 0, st, a);
}

// I tile: 64 output channels when the direction has at most 64, else 128.
static inline int igemm_bi(int ni) { return ni <= 64 ? 64 : 128; }

template <typename T, int DIR>
static hipError_t igemm_launch(IgArgs &a, int mj, int zdim, bool vi, bool vj, hipStream_t st) {
    const int bi = igemm_bi(a.NI);
    a.tiles_i = (a.NI + bi - 1) / bi;
    const int tiles_j = (mj + 127) / 128;
    const dim3 grid((unsigned)(a.tiles_i * tiles_j), 1, (unsigned)zdim);
    if (bi == 64)
        igemm_dispatch<T, DIR, 64>(a, grid, vi, vj, st);
    else
        igemm_dispatch<T, DIR, 128>(a, grid, vi, vj, st);
    return hipGetLastError();
}

// Tile configuration of the pipelined kernel: BI x BJ output tile, waves per block,
// LDS stages.
struct Igemm2Tile {
    int bi, bj, nw, ns;
};

// Relative time of `blocks` blocks on 256 CUs that hold two each: a full round of two per CU
// counts 1; a last round takes 0.6 when it gives no CU a second block (a block that has a CU to
// itself runs about 1.6 times as fast as one that shares it), more as second blocks come in.
static inline double round_cost(int64_t blocks) {
    const double f = (double)(blocks % 512) / 512.0;
    const double tail = f == 0.0 ? 0.0 : (f <= 0.5 ? 0.6 : std::min(1.0, 0.6 + 1.6 * (f - 0.5)));
    return (double)(blocks / 512) + tail;
}

// Chosen from sweeps over convolution layer shapes on MI355X.  Two 4-wave blocks share each CU.
// The copies into LDS (64 bytes per clock and CU) and the fragment reads out of it bound these
// kernels, so wide tiles pay as soon as there are blocks to fill the CUs:
//  * multiples of 128 channels with at least one 128 x 128 block per CU: 128-channel tiles.  Over
//    more than one round the row side is 128, 160 or 192 by round_cost times the tile's relative
//    time (1, 1.15, 1.4 for 1, 1.25, 1.5 times the work).  3 x 3, 56 x 56 x 256, batch 64, forward: 128 rows
//    242 us (6.1 rounds), 160 210 (4.9), 192 223 (4.1); 28 x 28 x 512, batch 64: 238, 210 and 230; input
//    gradient 256, 224, 248; 35 x 35 x 256 -> 384, batch 37: 94, 78, 85 and (input gradient) 95, 106, 76.
//  * multiples of 192 likewise (AlexNet conv2 forward: 76 -> 64 us);
//  * otherwise 64-channel tiles: 64 x 128, or 64 x 64 with three LDS stages up to 256 blocks, where
//    64 x 128 leaves every CU with one block whose barriers and copies nothing overlaps (17 x 17,
//    160 -> 192, 1 x 7, batch 32: forward 12.9 -> 12.0 us, 28 x 28 x 192 -> 96, 1 x 1, batch 8: 6.7 -> 5.7; over
//    random shapes 0.78-0.96 of the time), or 320 with reductions (per split or stride phase) below 1024
//    (0.91-0.97; from 1024 on 0.8-1.3: 40 x 21 x 21 x 80 <- 120, 7 x 7, 52.0 -> 68.1).
// kred: reduction elements of the whole product.
static inline Igemm2Tile igemm2_tiles(int ni, int mj, int zdim, int64_t kred) {
    const int64_t blocks_j = (int64_t)((mj + 127) / 128) * zdim;
    if (ni % 128 == 0 && (ni / 128) * blocks_j >= 256) {
        // 128-row tiles that leave most CUs with one block (AlexNet conv4/conv5: 338 blocks)
        // spread better as 96-row tiles, still within one round of two blocks per CU
        const int64_t b128 = (ni / 128) * blocks_j, b96 = (ni / 128) * (int64_t)((mj + 95) / 96) * zdim;
        // (not for a single row of tiles: 96-row tiles would leave most of the second row empty)
        if (b128 < 448 && b96 <= 512 && mj > 128) return {128, 96, 4, 2};
        Igemm2Tile best{128, 128, 4, 2};
        if (b128 <= 512) return best;
        double least = round_cost(b128);
        for (const auto &[bj, rel] : {std::pair{160, 1.15}, std::pair{192, 1.4}}) {
            const double c = rel * round_cost((ni / 128) * (int64_t)((mj + bj - 1) / bj) * zdim);
            if (c < least) {
                least = c;
                best.bj = bj;
            }
        }
        return best;
    }
    if (ni % 192 == 0 && (ni / 192) * blocks_j >= 256) {
        // 96-row J tiles when they fill the last round of two blocks per CU better: the same
        // operand reuse per byte (192 x 96 tiles read 64 flop per copied byte, 96 x 48 wave
        // tiles 32 per LDS byte, as 128 x 128 tiles do) in more, smaller blocks (AlexNet conv2
        // forward, 93312 pixels: 729 blocks of 128 rows fill 71 % of two rounds, 972 of 96
        // rows 95 %; 73.4 -> 71.9 us back to back)
        const int64_t b128 = (ni / 192) * blocks_j, b96 = (ni / 192) * (int64_t)((mj + 95) / 96) * zdim;
        auto fill = [](int64_t b) { return (double)b / (double)(((b + 511) / 512) * 512); };
        if (zdim == 1 && fill(b96) > fill(b128) + 0.05) return {192, 96, 4, 2};
        return {192, 128, 4, 2};
    }
    if ((int64_t)((ni + 63) / 64) * blocks_j <= (kred < 1024 * zdim ? 320 : 256)) return {64, 64, 4, 3};
    return {64, 128, 4, 2};
}

// At most 32 output rows (channels) on the I side: 32-row tiles, which keep every MFMA row in use
// (a 64-row tile would compute half or more of its rows for nothing).
static inline Igemm2Tile igemm2_tiles_narrow(int ni, int mj, int zdim, int64_t kred) {
    if (ni <= 32) return {32, 128, 4, 2};
    return igemm2_tiles(ni, mj, zdim, kred);
}

// fp32 tiles.  The fp32 matrix rate is a sixteenth of bf16's, so small tiles already keep the
// matrix cores busy (a 32 x 32 wave tile takes 1024 matrix cycles per K tile against 64 cycles of
// its own LDS reads): 64 x 64 tiles; 32 x 64 where 64-row tiles would compute a sixth or more of
// their rows for nothing (at most 32 channels, 96, 160) or give fewer blocks than CUs; 32 x 32 where
// 32 x 64 gives fewer.  16 x 28 x 28 x 96 -> 128, 3 x 3: forward 36 us with 64 x 64, 64 x 128 or 128 x 64
// tiles, 64 with 128 x 128 (register-staged kernel: 80); its input gradient 44 us with 32 x 64, 51 with
// 64 x 64 (register-staged kernel with its separate ReLU backward: 106).  8 x 14 x 14 x 256, 3 x 3: 55 us
// with 64 x 64 (100 blocks), 37 with 32 x 64, 35 with 32 x 32; 1 x 28 x 28 x 96 -> 64: 23, 16, 12.
static inline Igemm2Tile igemm2_tiles_f32(int ni, int mj, int zdim) {
    const int r32 = (ni + 31) / 32 * 32, r64 = (ni + 63) / 64 * 64;
    const int64_t bj = (int64_t)((mj + 63) / 64) * zdim;
    if ((r64 - r32) * 6 < r64 && r64 / 64 * bj >= 256) return {64, 64, 4, 3};
    return {32, r32 / 32 * bj < 256 ? 32 : 64, 4, 3};
}

// Whether the blocks of each stride phase of an input gradient are dealt to all XCDs.  Renumbered as a
// whole, an XCD runs blocks of one or two phases, and the phases' work is unequal: of a 1 x 1 filter's
// four at stride 2 one has the tap and three none, of a 3 x 3 filter's they have 4, 2, 2 and 1.  By phase
// every XCD has a part of each, but reads every phase's filter rows, which pays unless they outgrow its
// 4 MiB of L2 over only a round of blocks (strided input gradients at stride 2, by phase against whole:
// over 512 blocks 0.5-0.9 of the time, up to 1.04 with 7 x 7 filters over 16 MiB; 128-512 blocks 0.77-0.97
// with smaller filters, 0.97-1.1 with larger; below 128 blocks, or 256 where the phases differ by less
// than half (5 x 5, 7 x 7), 0.97-1.2: there each block has a CU to itself either way).
static inline int igemm2_by_phase(const IgArgs &a, int64_t blocks, int es) {
    const int most = ((a.KH + a.sh - 1) / a.sh) * ((a.KW + a.sw - 1) / a.sw) * a.sh * a.sw;
    if (a.k_split > 0 || most == a.KH * a.KW) return 0;       // (one phase, or equal ones)
    const int64_t filter = (int64_t)a.KH * a.KW * a.C * a.K * es;
    const int least = 2 * most >= 3 * a.KH * a.KW ? 128 : 256;
    return blocks > 512 || (blocks >= least && filter < (4 << 20)) ? 1 : 0;
}

template <typename T, int DIR, int BI, int BJ, int NW, int NS>
static void igemm2_go(const IgArgs &a, dim3 grid, hipStream_t st) {
    hipLaunchKernelGGL((igemm2_kernel<T, DIR, BI, BJ, NW, NS>), grid, dim3(NW * 64), 0, st, a);
}

template <int DIR>
static bool igemm2_launch_f32(IgArgs &a, int mj, int zdim, const Igemm2Tile &t, hipStream_t st) {
    a.tiles_i = (a.NI + t.bi - 1) / t.bi;
    const dim3 grid((unsigned)(a.tiles_i * ((mj + t.bj - 1) / t.bj)), 1, (unsigned)zdim);
    if (t.nw != 4 || t.ns != 3) return false;
    if (DIR == DIR_BWD_DATA) a.xcd_order = 1 + igemm2_by_phase(a, (int64_t)grid.x * grid.z, 4);
    if (t.bi == 64 && t.bj == 64) { igemm2_go<float, DIR, 64, 64, 4, 3>(a, grid, st); return true; }
    if (t.bi == 32 && t.bj == 64) { igemm2_go<float, DIR, 32, 64, 4, 3>(a, grid, st); return true; }
    if (t.bi == 32 && t.bj == 32) { igemm2_go<float, DIR, 32, 32, 4, 3>(a, grid, st); return true; }
    return false;
}

// Launches one of the compiled configurations; false if t is not one of them.  (96- and 160-row
// J tiles, 192-row ones and 192-channel tiles are forward and bwd-input only: the filter gradient
// keeps both operands k-major, with more address registers per copy, and spills there.)
template <int DIR>
static bool igemm2_launch(IgArgs &a, int mj, int zdim, const Igemm2Tile &t, hipStream_t st) {
    a.tiles_i = (a.NI + t.bi - 1) / t.bi;
    const int tiles_j = (mj + t.bj - 1) / t.bj;
    const dim3 grid((unsigned)(a.tiles_i * tiles_j), 1, (unsigned)zdim);
    if (t.nw != 4) return false;
    if (DIR == DIR_BWD_DATA) a.xcd_order = 1 + igemm2_by_phase(a, (int64_t)grid.x * grid.z, 2);
    const int key = t.bi * 10000 + t.bj * 10 + t.ns;
    switch (key) {
    case 321282: igemm2_go<bf16_t, DIR, 32, 128, 4, 2>(a, grid, st); return true;
    case 640643: igemm2_go<bf16_t, DIR, 64, 64, 4, 3>(a, grid, st); return true;
    case 641282: igemm2_go<bf16_t, DIR, 64, 128, 4, 2>(a, grid, st); return true;
    case 1281282: igemm2_go<bf16_t, DIR, 128, 128, 4, 2>(a, grid, st); return true;
    }
    if constexpr (DIR == DIR_FWD) {          // (64 x 192: the row bands of a pool inside the convolution)
        if (key == 641922) { igemm2_go<bf16_t, DIR, 64, 192, 4, 2>(a, grid, st); return true; }
    }
    if constexpr (DIR != DIR_BWD_FILTER) {
        switch (key) {
        case 1281283: igemm2_go<bf16_t, DIR, 128, 128, 4, 3>(a, grid, st); return true;
        case 1280962: igemm2_go<bf16_t, DIR, 128, 96, 4, 2>(a, grid, st); return true;
        case 1281602: igemm2_go<bf16_t, DIR, 128, 160, 4, 2>(a, grid, st); return true;
        case 1281922: igemm2_go<bf16_t, DIR, 128, 192, 4, 2>(a, grid, st); return true;
        case 1920962: igemm2_go<bf16_t, DIR, 192, 96, 4, 2>(a, grid, st); return true;
        case 1921282: igemm2_go<bf16_t, DIR, 192, 128, 4, 2>(a, grid, st); return true;
        }
    }
    return false;
}

// The kernel with the element-wise epilogue (RAG): the rule's tiles, of those compiled for it.
template <typename T>
static inline Igemm2Tile rag_tiles(int ni, int mj, int zdim, int64_t kred) {
    if constexpr (sizeof(T) == 4) {
        return Igemm2Tile{64, 64, 4, 3};
    } else {
        const Igemm2Tile t = igemm2_tiles(ni, mj, zdim, kred);
        return t.bi == 64 ? t : Igemm2Tile{128, 128, 4, 2};
    }
}

template <typename T, int DIR>
static hipError_t igemm2_launch_rag(IgArgs &a, int mj, int zdim, const Igemm2Tile &t, hipStream_t st) {
    a.tiles_i = (a.NI + t.bi - 1) / t.bi;
    const dim3 grid((unsigned)(a.tiles_i * ((mj + t.bj - 1) / t.bj)), 1, (unsigned)zdim), block(256);
    if (DIR == DIR_BWD_DATA) a.xcd_order = 1 + igemm2_by_phase(a, (int64_t)grid.x * grid.z, sizeof(T));
    if (t.bi == 64 && t.bj == 64)
        hipLaunchKernelGGL((igemm2_kernel<T, DIR, 64, 64, 4, 3, true>), grid, block, 0, st, a);
    else if constexpr (sizeof(T) == 2) {
        if (t.bi == 64)
            hipLaunchKernelGGL((igemm2_kernel<T, DIR, 64, 128, 4, 2, true>), grid, block, 0, st, a);
        else
            hipLaunchKernelGGL((igemm2_kernel<T, DIR, 128, 128, 4, 2, true>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}

// Split-K for GEMMs with few output tiles (fully connected layers at small batch): the
// reduction is cut into ranges of whole 64-wide K tiles, one per blockIdx.z, so that about 256
// blocks run, each range keeping at least 8 K tiles.  Returns the number of ranges (1: no split)
// and sets k_split to the range length in reduction elements.
//
// Weight streams (multiples of 128 channels): at most 256 blocks, so that each CU runs one of
// 128 x 128 with three LDS stages (igemm2_tiles_split) and two K tiles of copies in flight; with
// two stages one tile in flight per CU held the weights of 9216 -> 4096 at batch 128 to 2.3 TB/s.
// That layer, weights from HBM: forward 33.5 -> 25.4 us, input gradient 34.1 (288 blocks) -> 26.5 (216).
static inline int gemm_split_plan(int ni, int mj, int64_t kred, int *k_split) {
    const int64_t blocks = (int64_t)((ni + 127) / 128) * ((mj + 127) / 128);
    const int64_t ktiles = (kred + 63) / 64;
    int64_t want = (256 + blocks - 1) / blocks;
    if (ni % 128 == 0 && 256 / blocks >= 2 && 256 / blocks * blocks >= 192) want = 256 / blocks;
    const int64_t sp = std::min<int64_t>(want, ktiles / 8);
    *k_split = 0;
    if (blocks >= 128 || sp < 2) return 1;
    const int64_t per = (ktiles + sp - 1) / sp;
    *k_split = (int)(per * 64);
    return (int)((ktiles + per - 1) / per);
}

// Tiles of a split reduction: one 128 x 128 block per CU where the split gives about that many.
static inline Igemm2Tile igemm2_tiles_split(int ni, int mj, int sp, int64_t kred) {
    const int64_t blocks = (int64_t)((ni + 127) / 128) * ((mj + 127) / 128) * sp;
    if (ni % 128 == 0 && blocks >= 192 && blocks <= 256) return {128, 128, 4, 3};
    return igemm2_tiles_narrow(ni, mj, sp, kred);
}

// Bytes from the first element of a pixel-major operand (es bytes per element) to the end of its
// last pixel's channels.
static inline int64_t span_bytes(int64_t pixels, int64_t stride, int64_t ch, int64_t es = 2) {
    return pixels > 0 ? ((pixels - 1) * stride + ch) * es : 0;
}

// The pipelined kernel addresses each operand with 32-bit byte offsets (offsets from 2^31
// up read as zeros) and keeps masks of a filter's valid rows and columns in 31 bits.
// Records the spans when they fit.
static inline bool igemm2_fits(IgArgs &a, int64_t span_i, int64_t span_j) {
    constexpr int64_t kLim = int64_t(1) << 31;
    if (span_i >= kLim || span_j >= kLim || a.KH > 31 || a.KW > 31) return false;
    a.bytes_i = (uint32_t)span_i;
    a.bytes_j = (uint32_t)span_j;
    return true;
}

static inline void fill_geom(IgArgs &a, const ConvShape &s) {
    a.N = s.N; a.H = s.H; a.W = s.W; a.C = s.C;
    a.OH = s.OH; a.OW = s.OW; a.K = s.K;
    a.KH = s.KH; a.KW = s.KW; a.sh = s.sh; a.sw = s.sw; a.pt = s.pt; a.pl = s.pl;
    a.dC.init((uint32_t)s.C);
    a.dKW.init((uint32_t)s.KW);
    a.dOW.init((uint32_t)s.OW);
    a.dOH.init((uint32_t)s.OH);
    a.dK.init((uint32_t)s.K);
    a.beta = 0.f;
    a.bias = nullptr;
    a.xcd_order = 1;
    a.ni_store = 0;
    a.k_split = 0;
    a.split_stride = 0;
    a.bytes_i = a.bytes_j = 0;
    a.relu_y = nullptr;
    a.db_part = nullptr;
    a.db_rows = 0;
    a.band_rows = a.band_step = a.bands_per_img = 0;
    a.pool_y = nullptr;
    a.pool_taps = nullptr;
    a.pkh = a.pkw = a.psh = a.psw = a.pOH = a.pOW = a.pool_rows = 0;
    a.pool_ys = 0;
}

}  // namespace tfk
