// Which per-product kernel serves a layer call: channel lanes or the product list.
//
// Both skip products whose activation is zero, but not alike: the time of the channel lanes follows the number of products, the
// list also has a chain of latencies per ten taps and work per tap and pixel that is there whatever the activations are.
// How many of them are zero is not known on the host, and with a budget map neither is the number of samples.  So the rule
// compares the estimates at both ends, a quarter of the activations not zero and all of them, and departs from the plain
// answer - channel lanes for dense layers that fill at least half of the lanes of their last block (or pack it for four or eight
// pixels, with three quarters of the weights live), else the list - only if
// the other kernel is not slower at either end by more than 15 % and faster by 5 % in the mean of the two.  (Lanes packed for
// two pixels have to be 5 % faster at either end: a tap is skipped there only if both pixels have a zero, so what they gain
// depends most on what the host does not know.  3x3 24->20 on 3360 pixels, S = 32, lanes : list, estimates 95:96 and 194:251: list.)
// 3x3 on 64 channels, 4704 pixels, lanes : list in us, 8 channels, S = 4: 59:131 with a quarter, 188:229 with all (lanes); S = 8:
// 96:140 and 331:255 (list); 70 channels, S = 8: 177:292, 644:691 (lanes); 37->70, 5x5, 324 pixels, S = 10: 71:504 with half (lanes).
// Host code only (no HIP types), so that the rule can be tested against measured times without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace psb {

struct LayerWork {
    int K, OC;
    int64_t n_live;             // live weights of the layer
    double pixels;              // output pixels of the call
    int blocks;                 // generator blocks per product; with a budget map: at most
    bool budget_map;
    int lane_chunks, lane_taps; // channel lanes: chunks of the tap reduction, taps per chunk
    int list_channels;          // product list: channels of a workgroup, and its pixels
    int list_pixels, list_taps; // ... and live taps per chunk
    int packed_pixels = 0;      // channel lanes: pixels of a packed ticket of the last channel block (0: none)
};

// The estimates, in us, with the share `density` of the activations not zero and `blocks` generator blocks per product.  Their
// coefficients are fitted to 1032 layers at three densities each (1 to 512 channels, 1x1 to 5x5, 10 to 25000 pixels, 1 to 64 samples,
// 32 and 7 bits, budget maps): the root mean square of the relative error is 9 % for the lanes, 13 % for the list.

// Channel lanes: a ticket (one pixel, 64 channels, a chunk of taps) takes 0.24 us of a SIMD, and 58 ns per generator call of its
// wave; the last ticket of a wave runs alone.  A split reduction has a second launch.  A packed ticket (several pixels of the last
// channels) takes another 0.075 us a pixel, and a call wherever one of its pixels has an activation.
inline double channel_lane_us(const LayerWork& w, double density, double blocks, int n_cus)
{
    const bool split = w.lane_chunks > 1, packed = w.packed_pixels > 1;
    const double call_us = 0.061 * w.lane_taps * blocks;
    const double plain_blocks = (w.OC + 63) / 64 - (packed ? 1 : 0), per_simd = w.lane_chunks / (4.0 * n_cus);
    double us = 4.9 + (split ? 3.9 : 0.0) + w.pixels * plain_blocks * per_simd * (0.24 + 0.925 * density * call_us);
    double last = plain_blocks > 0 ? density : 0.0;
    if (packed) {
        double none = 1.0 - density;                     // a tap has no activation at any of the 2, 4 or 8 pixels
        for (int n = 1; n < w.packed_pixels; n *= 2) none *= none;
        const double any = 1.0 - none;
        us += std::ceil(w.pixels / w.packed_pixels) * per_simd * (0.24 + 0.075 * w.packed_pixels + 0.925 * any * call_us);
        last = any;
    }
    return std::max(us + 1.3 * last * call_us, split ? 14.5 : 12.0);                          // what launching takes
}

// Product list: a workgroup walks its live taps ten at a time, up to eight blocks a pass; a chunk takes 1.9 us alone on its CU (table,
// gather, compaction, barriers one after the other) and its share of samples on top, every further workgroup of the CU 0.08 us and
// the work itself.  Calls with a budget map have no tables: three times the work per sample.
inline double product_list_us(const LayerWork& w, double density, double blocks, int n_cus)
{
    const double taps = (double)w.n_live / w.OC;
    const double columns = std::ceil(w.pixels / w.list_pixels);
    const double filled = w.pixels / (w.list_pixels * columns);
    // workgroups per CU (one or two over a full row do not show: 2.004 measures as 2)
    const double more = std::max(0.0, std::ceil(columns * ((w.OC + w.list_channels - 1) / w.list_channels) / n_cus - 0.25) - 1.0);
    const double passes = w.budget_map ? 1.0 : std::ceil(blocks / 8.0);
    const double chunks = w.list_channels * std::ceil(taps / w.list_taps);
    const double samples = density * filled * blocks * (w.budget_map ? 3.0 : 1.0);
    const double us = 3.0 + chunks * passes * (1.87 + 0.083 * more) +
                      w.list_channels * taps * (samples * (0.128 + 0.060 * more) + passes * 0.024 * more);
    return std::max(us, 12.0);
}

inline bool prefer_channel_lanes(const LayerWork& w, int n_cus)
{
    const int last = w.OC % 64;
    const bool plain = 2 * w.n_live >= (int64_t)w.OC * w.K && (last == 0 || last >= 32 || w.OC >= 256 ||
                                                                     (w.packed_pixels > 2 && 4 * w.n_live >= 3 * (int64_t)w.OC * w.K));
    auto list_over_lanes = [&](double density, double blocks) {
        return std::log(product_list_us(w, density, blocks, n_cus) / channel_lane_us(w, density, blocks, n_cus));
    };
    const double sparse = list_over_lanes(0.25, w.budget_map ? 1.0 : w.blocks), full = list_over_lanes(1.0, w.blocks);
    const double sign = plain ? -1.0 : 1.0;               // > 0: the other kernel is the faster one
    const bool two_pixels = !plain && w.packed_pixels == 2;
    const bool other = std::min(sign * sparse, sign * full) >= (two_pixels ? 0.05 : -std::log(1.15)) && sign * (sparse + full) > 0.1;
    return plain != other;
}

}  // namespace psb
