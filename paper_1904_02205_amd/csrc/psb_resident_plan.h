// How k_conv3x3_resident cuts a layer, and which layers it takes.  Host code only (no HIP types), so that the cuts can be tested
// without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace psb {

constexpr int kResidentWaves = 8;
constexpr int kResidentSlots = 1024;        // window slots at most
constexpr int kResidentEntry = 16;          // bytes of a PixelEntry
constexpr int kResidentLds = 156 * 1024;    // dynamic LDS at most (the CU has 160 KB)

// How the launcher cuts a layer.
struct ResidentPlan {
    int log_wo, log_wp, log_wk;             // waves of a workgroup: channel groups x pixel parts x reduction parts
    int ng;                                 // pixel groups of a wave
    int part;                               // pixels of a wave's part, at most 16 ng, a multiple of 4
    // 16-byte words of a quarter of a 64-channel chunk in LDS, a multiple of 16: a wave's 16-byte reads then take 4.8 cycles of
    // the LDS (8.3 where a group of pixels crosses a row), with an odd multiple of 8 they take 8.3 (12.2)
    int slots_pad;
    unsigned px_tiles, oc_tiles;
    uint32_t inv_oc_tiles;                  // inverse_of(oc_tiles), set by the launcher
    int by_channels;                        // an XCD takes an eighth of the channel tiles instead of the pixel tiles
    int lds_window;                         // offset of the window in LDS, behind the tables of the tile's pixels
    int lds_zero;                           // offset of 16 zero bytes
    int lds_res;                            // offset of the residual, [channel group][pixel of the tile][16], if it is staged (else 0)
    int lds_bytes;
};

// A 3 x 3 layer with unit stride and one pixel of padding, as the plan sees it.
struct ResidentLayer {
    int64_t npix;                           // output pixels of the call, N H W
    int H, W, OC;
    int blocks;                             // of 32 input channels
    int planes, n_seg;                      // digit planes (2 or 3); segments of the sample axis, 0: no announced levels
    int half_tiles;                         // of a wave in the kernels that take the layer otherwise, shared_half_tiles()
    bool residual;                          // a residual that a workgroup can stage: int8, blocked, on a 16-byte address
};

// The longest window of `tile` consecutive pixels: as for k_conv3x3_window.
inline int64_t resident_slots(int64_t tile, int H, int W)
{
    const int64_t rows = (tile + W - 2) / W, images = (tile + (int64_t)H * W - 2) / ((int64_t)H * W);
    return tile - 1 + rows + images * (W + 1) + 2 * (W + 1) + 3;
}

// The cut of a layer with the smallest estimate, or false: not a layer for this kernel.
inline bool resident_plan(const ResidentLayer& l, int n_cus, ResidentPlan& best)
{
    // An instruction takes 64 channels: with one or three blocks of 32 half or a quarter of them are padding, which the kernels of
    // 32 channels do not multiply.  Over random layers of 1 to 64 images, times as fast as in those: 1 block 0.85 to 1.1, 3 blocks 0.94
    // to 1.46; the others below.
    if (l.blocks == 1 || l.blocks == 3) return false;
    const int64_t npix = l.npix;
    const int planes = l.planes;
    if (npix * ((l.OC + 31) / 32 * 32) >= (1ll << 31)) return false;    // activations are addressed with 32-bit offsets
    const int n_oc16 = 2 * ((l.OC + 31) / 32), n_chunks = (l.blocks + 1) / 2, steps = 9 * n_chunks;
    double best_us = 1e30;
    for (int log_wo = 0; log_wo <= 3; ++log_wo)
        for (int log_wk = 0; log_wk + log_wo <= 3; ++log_wk) {
            const int log_wp = 3 - log_wo - log_wk;
            if ((1 << log_wo) > n_oc16 || steps < 2 << log_wk) continue;
            const int64_t oc_tiles = (n_oc16 + (1 << log_wo) - 1) >> log_wo;
            for (int ng : {4, 7, 13}) {
                if (ng > 7 && (log_wk > 0 || l.n_seg > 0)) continue;         // (segments would spill)
                // The fewest rounds of one workgroup per CU, and inside them the smallest equal parts.  Not more than two: nothing of a
                // round lies under the next one, which the kernels of two workgroups per CU do better (384->96 at 28x95, batch 16,
                // five rounds: 64.6 us against 40.2).
                const int64_t most = 16 * ng;
                int64_t rounds = std::max<int64_t>(1, ((npix + (most << log_wp) - 1) / (most << log_wp) * oc_tiles + n_cus - 1) / n_cus);
                int64_t part = 0, px_tiles = 0;
                for (; rounds <= 2; ++rounds) {
                    const int64_t tiles = rounds * n_cus / oc_tiles;
                    if (tiles == 0) continue;
                    part = (((npix + tiles - 1) / tiles + (1 << log_wp) - 1) >> log_wp);
                    part = (part + 3) / 4 * 4;
                    if (part <= most) break;
                }
                // microseconds of a round: start and end, matrix instructions of two waves per SIMD, the end of a wave; then the window
                const double least_us = rounds * (4.0 + (double)((steps + (1 << log_wk) - 1) >> log_wk) * ng * planes * 2 * 16 / 2400.0 / 0.7 +
                                                  0.15 * ng / (1 << log_wk) + 0.05 * ng * (log_wk > 0));
                if (rounds > 2 || least_us >= best_us) continue;
                px_tiles = (npix + (part << log_wp) - 1) / (part << log_wp);
                const int64_t slots = resident_slots(part << log_wp, l.H, l.W);
                const int64_t pad = (slots + 15) / 16 * 16;
                const int64_t window = pad * 64 * n_chunks, meet = (int64_t)(kResidentWaves >> log_wk) * ng * ((1 << log_wk) - 1) * 1024;
                const int64_t table = (part << log_wp) * kResidentEntry;
                // the residual behind them, where there is room for it
                const int64_t res_at = table + std::max(window + 16, meet), res = (part << log_wp << log_wo) * 16;
                const bool stage_res = ng > 7 && l.residual && res_at + res <= kResidentLds;
                const int64_t lds = stage_res ? res_at + res : res_at;
                if (slots > kResidentSlots || lds > kResidentLds) continue;
                const double us = least_us + rounds * (double)window / 60000.0;
                if (us < best_us) {
                    best_us = us;
                    best.log_wo = log_wo; best.log_wp = log_wp; best.log_wk = log_wk; best.ng = ng; best.part = (int)part;
                    best.slots_pad = (int)pad; best.px_tiles = (unsigned)px_tiles; best.oc_tiles = (unsigned)oc_tiles;
                    best.lds_window = (int)table; best.lds_zero = (int)(table + window); best.lds_res = stage_res ? (int)res_at : 0;
                    best.lds_bytes = (int)lds;
                }
            }
        }
    if (best_us >= 1e30) return false;
    // Equal shares of a layer need not be whole groups of pixels or blocks of channels, and LDS may not hold the window of larger
    // ones: then a part of the matrix instructions multiplies padding.  What counts is their number on the busiest CU, against that of
    // the kernels of 32 channels x 128 or 256 pixels.  Random layers, times as fast as in those, by the quotient theirs / ours: one
    // round, below 0.7 0.84 to 1.10 (five layers, four of them slower; 768->128 at 56x56, one image, parts of 16 pixels in four groups:
    // 35.6 us against 29.7), from 0.7 on 0.95 to 2.5 (6234 layers, mean 1.33); two rounds, below 0.9 0.81 to 1.10 (53 layers, 40 of them
    // slower: 256->128 at 10x93, batch 64, parts of 120 pixels in thirteen groups: 77.0 us against 62.1), from 0.9 on 0.94 to 1.38 (194
    // layers, mean 1.14) ...
    const int64_t rounds = ((int64_t)best.px_tiles * best.oc_tiles + n_cus - 1) / n_cus, wg_pixels = 128 * l.half_tiles;
    const int64_t ours = rounds * kResidentWaves * best.ng * ((steps + (1 << best.log_wk) - 1) >> best.log_wk);
    const int64_t their_wgs = (npix + wg_pixels - 1) / wg_pixels * (n_oc16 / 2);
    const int64_t theirs = (their_wgs + n_cus - 1) / n_cus * 8 * l.half_tiles * 9 * l.blocks;
    if (10 * theirs < (rounds == 1 ? 7 : 9) * ours) return false;
    // ... but for two forms that two rounds do not pay for: parts of the reduction that meet in LDS, which the second round waits for
    // (69 layers, 0.89 to 1.23, mean 1.02, a third of them slower; 256->16 at 14x106, batch 64: 29.3 us against 26.0), and four groups of
    // two planes, whose operands take all that L2 and LDS deliver to a CU (twelve layers, 0.86 to 0.99; 640->512 at 56x56, two images:
    // 121.9 us against 108.2).
    if (rounds > 1 && (best.log_wk > 0 || (best.ng == 4 && planes == 2))) return false;
    const int64_t n_steps = (int64_t)9 * l.blocks;
    best.by_channels = best.oc_tiles % 8 == 0 && (int64_t)n_oc16 * 16 * n_steps * 32 * planes > 2 * npix * 32 * l.blocks;
    return true;
}

}  // namespace psb
