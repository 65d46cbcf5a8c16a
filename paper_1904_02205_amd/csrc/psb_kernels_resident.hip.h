// Shared-filter mode, 3 x 3 layers with unit stride and one pixel of padding: the whole input window of a pixel tile in LDS.
//
// A workgroup of eight waves keeps every input channel of the pixels its tile touches in LDS - staged once, one barrier -
// and after that its waves run on their own: the weight operands come straight from L2, each wave's own, a step ahead in
// registers, and no barrier or staging interrupts the matrix instructions.  A wave holds 16 output channels x NG groups of
// 16 pixels (v_mfma_i32_16x16x64_i8: 64 channels of a tap at a time), so a weight operand is used NG times and an
// activation operand P times (P digit planes); per matrix instruction of 16 cycles that is 1 KB / NG from L2 and 1 KB / P
// from LDS.  The eight waves are wo groups of channels x wp parts of the pixels x wk parts of the reduction, whose sums
// meet in LDS at the end.  Fine tiles (16 x 16) are the point: the launcher cuts the layer so that every CU gets the same
// number of them, where tiles of 32 channels x 128 or 256 pixels leave a second, half empty round.
//
// Time stamps of a workgroup, batch 32, us - 64->64 at 56x56 (13 groups): staged 3.3, loop of the older / younger four waves
// 5.9 / 8.2, end of a wave 3.0; 128->128 at 28x28 and 256->256 at 14x14 (7 groups): 2.1, 7.0 / 9.2, 2.4.  The matrix instructions alone
// need 5.9 and 6.3 us of the loop at the 1.9 GHz the chip holds in it (2.4 without them).  A launch, in the kernel trace of a
// whole network pass: 23.3 us in k_conv3x3_window, 17.7 here (64->64); 18.6 and 16.1 (the later stages).  Without effect: weights
// and activations left out of the loop (-0.7 to -1.1 us), wave priorities, the residual requested a few steps before the end
// (it delays the weights behind it by as much).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "psb_kernels_shared.hip.h"
#include "psb_resident_plan.h"

namespace psb {

// What the waves of a workgroup need to know of a pixel of its tile, made once per workgroup: every wave would need some 40
// vector instructions for each of its groups otherwise.
struct PixelEntry {
    uint32_t slot;                          // its tap (0, 0) in the window
    uint32_t blocked;                       // offset of channel 0 in the blocked layout with the output's channel blocks
    uint32_t flat;                          // index of channel 0 in [N][OC][OH][OW]
    uint32_t to;                            // samples
};
static_assert(sizeof(PixelEntry) == kResidentEntry, "the plan reserves this much for an entry");

// Offsets of a lane's words of requantised activations: four channels of a pixel (blocked), or four pixels of one channel
// ([N][OC][OH][OW]; see tile_epilogue).  Words that do not exist have an offset beyond the tensor.
template <int NG, bool FULL, class At, class Exists>
__device__ __forceinline__ void word_offsets(const SharedParams& p, bool blocked, int oc_first, At at, Exists exists, uint32_t (&off)[NG])
{
    const uint32_t plane = (uint32_t)(p.OH * p.OW), j = threadIdx.x & 3u;
    if (blocked) {
        const uint32_t from_block = ((uint32_t)oc_first >> 5) * (uint32_t)p.OW * 32u + ((uint32_t)oc_first & 31u);
#pragma unroll
        for (int g = 0; g < NG; ++g) off[g] = exists(g) ? at(g).blocked + from_block : kOutOfRange;
    } else {
        const bool channel = FULL || oc_first + (int)j < p.OC;
#pragma unroll
        for (int g = 0; g < NG; ++g) off[g] = exists(g) && channel ? (at(g).flat & ~3u) + ((uint32_t)oc_first + j) * plane : kOutOfRange;
    }
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t word_buffer(const SharedParams& p, const int8_t* tensor, bool blocked)
{
    const uint32_t plane = (uint32_t)(p.OH * p.OW);
    return operand_buffer(tensor, (uint32_t)p.N * plane * (uint32_t)(blocked ? (p.OC + 31) & ~31 : p.OC));
}

// The end of a wave's tile: its sums u[g][i] - channel oc_first + i of pixel 16 g + col of its part - become accumulators and
// rescaled values, or requantised activations.  Flags are looked at once per kind of access and not once per group, and loads and
// stores of whole words go through range-checked buffers: with a branch around each of them this took twice the time of the
// matrix instructions of a layer of 64 channels.  A wave is alone or nearly alone on its SIMD here and issues an instruction
// every 2.3 ns, so what counts is their number.
// mine(g): this wave finishes group g.  at(g): the pixel's entry.  exists(g): this lane's pixel exists.  res_word: the words
// of res_i8, requested earlier, if they can be read as words.
template <int OUT, int NG, bool FULL, bool SEG, class Mine, class At, class Exists>
__device__ __forceinline__ void finish_tile(const SharedParams& p, const uint32_t (&u)[NG][4], int oc_first, const float (&mult)[4],
                                            const float (&bias)[4], uint32_t (&res_word)[NG], Mine mine, At at, Exists exists)
{
    const uint32_t plane = (uint32_t)(p.OH * p.OW), from_flat = (uint32_t)oc_first * plane;
    auto inverse = [](int to) { return to > 0 ? __fdiv_rn(1.0f, (float)to) : 0.0f; };
    const float inv_everywhere = SEG ? 0.0f : inverse(min(p.S, p.s_max));
    auto inv_of = [&](int g) { return SEG ? inverse((int)at(g).to) : inv_everywhere; };
    auto rescaled = [&](int g, int i) {                // the arithmetic of rescale()
        float r = __fmul_rn(__fmul_rn(__int2float_rn((int32_t)u[g][i]), mult[i]), inv_of(g));
        if (p.bias) r = __fadd_rn(r, bias[i]);
        return r;
    };
    auto each = [&](auto&& f) {                        // existing channels of existing pixels, with their flat index
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (!mine(g)) continue;                    // uniform
            if (exists(g)) {
                const uint32_t flat = at(g).flat + from_flat;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (FULL || oc_first + i < p.OC) f(g, i, flat + (uint32_t)i * plane);
            }
        }
    };
    if (p.acc) each([&](int g, int i, uint32_t o) { p.acc[o] = (int32_t)u[g][i]; });
    if (p.y) each([&](int g, int i, uint32_t o) { p.y[o] = rescaled(g, i); });
    if constexpr (OUT == kOutRequant) {
        // words of four channels of a pixel (blocked), or of four pixels of one channel ([N][OC][OH][OW]; see tile_epilogue)
        // The integers of requantize_one() as in tile_epilogue with fewer instructions: the gate is a lower bound of zero, or of hi
        // where that is below zero and every result is hi (the host keeps the scales for which it is not away), the bounds are
        // integers, so clamping before rounding gives the same (a NaN ends at the lower bound: the minimum of three), and adding
        // 1.5 * 2^23 rounds to the nearest integer, ties to even.
        const float lo = p.rq.relu ? __builtin_fminf(__builtin_fmaxf(p.rq.lo, 0.0f), p.rq.hi) : p.rq.lo;
        uint32_t word[NG];
        auto requantised = [&](auto res) {             // res(g, i): the residual
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (!mine(g)) continue;
                const float inv_s = inv_of(g);
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float t = __fmul_rn(__fmul_rn(__int2float_rn((int32_t)u[g][i]), mult[i]), inv_s);
                    t = __fadd_rn(__fadd_rn(t, bias[i]), res(g, i));
                    w[i] = __float_as_uint(__fadd_rn(__builtin_amdgcn_fmed3f(__fmul_rn(t, p.rq.inv_step), lo, p.rq.hi), 12582912.0f));
                    if (!FULL && oc_first + i >= p.OC) w[i] = 0;      // padding channels of the blocked layout
                }
                word[g] = __builtin_amdgcn_perm(w[1], w[0], 0x0c0c0400u) | __builtin_amdgcn_perm(w[3], w[2], 0x04000c0cu);
            }
        };
        if (p.rq.res_f32) {
            float res[NG][4];
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) res[g][i] = 0.0f;
            each([&](int g, int i, uint32_t o) { res[g][i] = p.rq.res_f32[o]; });
            requantised([&](int g, int i) { return res[g][i]; });
        } else if (p.rq.res_i8) {
            if (!(p.rq.res_blocked || p.quad_res)) {
#pragma unroll
                for (int g = 0; g < NG; ++g) res_word[g] = 0;
                each([&](int g, int i, uint32_t o) { res_word[g] |= (uint32_t)(uint8_t)p.rq.res_i8[o] << (8 * i); });
            } else if (!p.rq.res_blocked) {
#pragma unroll
                for (int g = 0; g < NG; ++g) res_word[g] = quad_transpose_bytes(res_word[g]);
            }
            requantised([&](int g, int i) { return __fmul_rn((float)(int8_t)(res_word[g] >> (8 * i)), p.rq.res_step); });
        } else {
            requantised([&](int, int) { return 0.0f; });
        }
        if (p.rq.out_blocked || p.quad_store) {
            const __amdgpu_buffer_rsrc_t rsrc = word_buffer(p, p.rq.x_out, p.rq.out_blocked != 0);
            uint32_t off[NG];
            word_offsets<NG, FULL>(p, p.rq.out_blocked != 0, oc_first, at, exists, off);
            if (!p.rq.out_blocked) {
#pragma unroll
                for (int g = 0; g < NG; ++g) word[g] = quad_transpose_bytes(word[g]);
            }
#pragma unroll
            for (int g = 0; g < NG; ++g)
                if (mine(g)) __builtin_amdgcn_raw_buffer_store_b32(word[g], rsrc, (int)off[g], 0, 0);
        } else {
            each([&](int g, int i, uint32_t o) { p.rq.x_out[o] = (int8_t)(word[g] >> (8 * i)); });
        }
    }
}

// P digit planes, NG groups of 16 pixels per wave; SEG: a budget map with announced levels (see SharedParams::n_seg).
// Every workgroup of the grid runs every barrier; a wave without channels or pixels only stages.
template <int P, int OUT, int NG, bool SEG>
__global__ void __launch_bounds__(kResidentWaves * 64, 2) k_conv3x3_resident(const SharedParams p, const ResidentPlan plan)
{
    touch_arguments<SharedParams, ResidentPlan>();
    constexpr bool kStageRes = OUT == kOutRequant && NG > 7;
    extern __shared__ v4i win[];                   // entries of the tile's pixels; [chunk of 64 channels][quarter of 16][slot]; zeros
    __shared__ __align__(16) float s_mult[128], s_bias[128];            // read four at a time
    int8_t* const lds = reinterpret_cast<int8_t*>(win);
    PixelEntry* const entries = reinterpret_cast<PixelEntry*>(win);      // [pixel of the tile]

    const int tid = (int)threadIdx.x, lane = tid & 63, wave = (int)uniform_u32((uint32_t)tid >> 6);
    const int col = lane & 15, quarter = lane >> 4;
    const int og = wave & ((1 << plan.log_wo) - 1);
    const int pp = (wave >> plan.log_wo) & ((1 << plan.log_wp) - 1);
    const int kp = wave >> (plan.log_wo + plan.log_wp);
    const uint32_t npix = (uint32_t)((int64_t)p.N * p.OH * p.OW);       // fits 32 bits (checked by the host)

    unsigned px_tile, oc_tile;
    if (plan.by_channels) {
        // oc_tiles is a multiple of 8 and the grid exact: XCD = workgroup mod 8 owns oc_tiles / 8 consecutive channel tiles
        const unsigned local = blockIdx.x >> 3, per_xcd = plan.oc_tiles >> 3;
        px_tile = local / per_xcd;
        oc_tile = (blockIdx.x & 7u) * per_xcd + (local - px_tile * per_xcd);
    } else {
        const unsigned at = xcd_contiguous(blockIdx.x, plan.px_tiles * plan.oc_tiles);
        if (at == 0xFFFFFFFFu) return;             // uniform over the workgroup, before any barrier
        px_tile = div_mod(at, plan.oc_tiles, plan.inv_oc_tiles, oc_tile);
    }
    const uint32_t tile = (uint32_t)plan.part << plan.log_wp;
    const uint32_t pix_first = px_tile * tile;
    const int CB = p.C_pad >> 5, n_chunks = (CB + 1) >> 1;
    const uint32_t W1 = (uint32_t)p.tW + 1u, H1 = (uint32_t)p.tH + 1u;
    const int oc16 = (int)(oc_tile << plan.log_wo) + og;                // this wave's 16 channels
    const int n_oc16 = 2 * ((p.OC + 31) >> 5);

    // weights: lane's row of the 16 x 64 operand inside the planes' [32 channels][16 of 32 input channels] operands
    const int8_t* const wblock = p.planes + (int64_t)min(oc16 >> 1, (n_oc16 >> 1) - 1) * p.n_ksteps * (kMaxPlanes * kPlaneStride);
    const uint32_t a_off = (uint32_t)((col + 16 * (oc16 & 1) + 32 * (quarter & 1)) * 16 + (quarter >> 1) * (kMaxPlanes * kPlaneStride));
    const int total_steps = 9 * n_chunks;                               // (chunk, tap), tap fastest
    const int s_begin = (total_steps * kp) >> plan.log_wk, s_end = (total_steps * (kp + 1)) >> plan.log_wk;
    // where a step's weights and activations are, stepped on the scalar unit
    struct Cursor { int tap; uint32_t weights, window; };
    auto cursor_at = [&](int s) {
        const int c = s / 9, t = s - 9 * c;
        return Cursor{t, (uint32_t)(t * CB + 2 * c) * (uint32_t)(kMaxPlanes * kPlaneStride), (uint32_t)(c * 4 * plan.slots_pad + t / 3 * (int)W1 + t % 3) * 16u};
    };
    const uint32_t tap_stride = (uint32_t)CB * (uint32_t)(kMaxPlanes * kPlaneStride), row_step = (W1 - 2u) * 16u;
    const uint32_t chunk_weights = 2u * (uint32_t)(kMaxPlanes * kPlaneStride) - 8u * tap_stride;
    const uint32_t chunk_window = (uint32_t)plan.slots_pad * 64u - (2u * W1 + 2u) * 16u;
    auto advance = [&](Cursor& k) {
        const bool next_chunk = k.tap == 8, next_row = k.tap == 2 || k.tap == 5;
        k.weights += next_chunk ? chunk_weights : tap_stride;
        k.window += next_chunk ? chunk_window : next_row ? row_step : 16u;
        k.tap = next_chunk ? 0 : k.tap + 1;
    };
    __amdgpu_buffer_rsrc_t w_rsrc = operand_buffer(wblock, (uint32_t)(p.n_ksteps + kStageSteps) * (kMaxPlanes * kPlaneStride));
    v4i a[2][P];
    auto fetch = [&](v4i (&dst)[P], const Cursor& k) {
#pragma unroll
        for (int b = 0; b < P; ++b) dst[b] = load_operand(w_rsrc, a_off, k.weights + (uint32_t)(b * kPlaneStride));
    };

    fetch(a[0], cursor_at(s_begin));               // first of all: nothing below depends on it until the barrier
    // rescale factors of the workgroup's channels, by the last waves
    const int f_at = tid - (kResidentWaves * 64 - 128), f_oc = (int)(oc_tile << plan.log_wo) * 16 + f_at;
    float f_mult = p.default_mult, f_bias = 0.0f;
    if (f_at >= 0 && f_oc < p.OC) {
        if (p.mult) f_mult = p.mult[f_oc];
        if (p.bias) f_bias = p.bias[f_oc];
    }

    // the window: slot s holds virtual position q_first + s (see k_conv3x3_window)
    auto virtual_position = [&](uint32_t pix, uint32_t& row, uint32_t& n, uint32_t& ox) {
        uint32_t oy;
        row = div_mod(pix, (uint32_t)p.OW, p.inv_OW, ox);
        n = div_mod(row, (uint32_t)p.OH, p.inv_OH, oy);
        return (row + n) * W1 + ox;                // (n H1 + oy) W1 + ox, H1 = OH + 1
    };
    const uint32_t pix_end = min(pix_first + tile, npix);
    uint32_t row_, n_, ox_;
    const uint32_t q_first = virtual_position(pix_first, row_, n_, ox_);
    const uint32_t n_slots = virtual_position(pix_end - 1u, row_, n_, ox_) - q_first + 2u * W1 + 3u;
    int8_t* const window = lds + plan.lds_window;
    {
        const __amdgpu_buffer_rsrc_t xt_rsrc = operand_buffer(p.xt, p.xt_bytes);
        const uint32_t half = (uint32_t)tid & 1u, cb_stride = (uint32_t)p.tW * 32u, quarter_bytes = (uint32_t)plan.slots_pad * 16u;
        for (uint32_t s = (uint32_t)tid >> 1; s < n_slots; s += kResidentWaves * 32) {     // two threads a slot
            uint32_t vc, rr;
            const uint32_t vr = div_mod(q_first + s, W1, p.inv_W1, vc);
            const uint32_t n = div_mod(vr, H1, p.inv_H1, rr);
            const bool ok = vc >= 1u && rr >= 1u && n < (uint32_t)p.N;
            const uint32_t from = ok ? (vr - n - 1u) * (uint32_t)(CB * p.tW) * 32u + (vc - 1u) * 32u + 16u * half : kOutOfRange;
            int8_t* to = window + half * quarter_bytes + s * 16u;
            auto stage = [&](auto count_c, int cb) {           // so many channel blocks with their loads in flight together
                constexpr int COUNT = decltype(count_c)::value;
                v4i v[COUNT];
#pragma unroll
                for (int i = 0; i < COUNT; ++i) v[i] = load_operand(xt_rsrc, cb + i < CB ? from : kOutOfRange, (uint32_t)(cb + i) * cb_stride);
#pragma unroll
                for (int i = 0; i < COUNT; ++i) *reinterpret_cast<v4i*>(to + (uint32_t)(cb + i) * 2u * quarter_bytes) = v[i];
            };
            int cb = 0;
            for (; cb + 8 <= 2 * n_chunks; cb += 8) stage(std::integral_constant<int, 8>{}, cb);
            for (; cb < 2 * n_chunks; cb += 2) stage(std::integral_constant<int, 2>{}, cb);
        }
        // Waves of many groups stage a residual in the blocked layout as well: requested at the end it would take 2.5 us, at the
        // same time in every workgroup and with nothing to hide it.  (With seven groups and fewer it is 0.9 us either way.)
        const __amdgpu_buffer_rsrc_t res_rsrc = word_buffer(p, kStageRes && plan.lds_res ? p.rq.res_i8 : p.xt, true);
        const int first16 = (int)(oc_tile << plan.log_wo), n16 = kStageRes && plan.lds_res ? min(1 << plan.log_wo, n_oc16 - first16) : 0;
        for (uint32_t i = (uint32_t)tid; i < tile; i += kResidentWaves * 64) {
            const uint32_t pix = min(pix_first + i, npix - 1u);       // beyond the layer: its last pixel, not stored
            PixelEntry e;
            uint32_t row, n, ox;
            e.slot = virtual_position(pix, row, n, ox) - q_first;
            e.blocked = (row * (uint32_t)((p.OC + 31) >> 5) * (uint32_t)p.OW + ox) * 32u;
            e.flat = pix + n * (uint32_t)(p.OC - 1) * (uint32_t)(p.OH * p.OW);
            int to;
            (void)shared_pixel_range(p, pix, to);
            e.to = (uint32_t)to;
            entries[i] = e;
            if constexpr (kStageRes) {
                v4i res[kResidentWaves];
#pragma unroll
                for (int j = 0; j < kResidentWaves; ++j)
                    if (j < n16)                                        // uniform
                        res[j] = load_operand(res_rsrc, e.blocked, (uint32_t)((first16 + j) >> 1) * (uint32_t)p.OW * 32u + (uint32_t)((first16 + j) & 1) * 16u);
#pragma unroll
                for (int j = 0; j < kResidentWaves; ++j)
                    if (j < n16) *reinterpret_cast<v4i*>(lds + plan.lds_res + ((uint32_t)j * tile + i) * 16u) = res[j];
            }
        }
        if (tid == 0) *reinterpret_cast<v4i*>(lds + plan.lds_zero) = v4i{0, 0, 0, 0};
        if (f_at >= 0) { s_mult[f_at] = f_mult; s_bias[f_at] = f_bias; }
    }
    const uint32_t part_at = (uint32_t)(pp * plan.part);                // inside the tile
    const bool active = oc16 < n_oc16 && pix_first + part_at < npix;    // wave-uniform
    // entry of this lane's pixel in group g; the part's last pixel where the part ends before
    auto entry_of = [&](int g) -> const PixelEntry& { return entries[part_at + (uint32_t)min(16 * g + col, plan.part - 1)]; };
    __syncthreads();
    uint32_t slot[NG];                             // offset of the pixel's tap (0, 0), this lane's quarter
#pragma unroll
    for (int g = 0; g < NG; ++g) slot[g] = (uint32_t)plan.lds_window + ((uint32_t)(quarter * plan.slots_pad) + entry_of(g).slot) * 16u;

    const int wk = NG > 7 ? 1 : 1 << plan.log_wk;
    if (!active) {
        if (wk > 1) { __syncthreads(); __syncthreads(); }               // those of the meeting below
        return;
    }
    v4i acc[NG][P];

    int n_seg = 1;
    for (int seg = 0; seg < n_seg; ++seg) {
        unsigned long long takes[SEG ? NG : 1];    // lanes whose pixel reaches this segment
        if constexpr (SEG) {
            if (seg == 0) n_seg = p.n_seg;
            bool any = false;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                takes[g] = __ballot((int)entry_of(g).to >= p.seg_level[seg]);
                any |= takes[g] != 0ull;
            }
            if (!any && seg > 0) break;            // levels nest (and the first pass clears the sums)
            w_rsrc = operand_buffer(wblock + (int64_t)seg * (int64_t)p.seg_stride, (uint32_t)(p.n_ksteps + kStageSteps) * (kMaxPlanes * kPlaneStride));
        }
        Cursor ahead = cursor_at(s_begin);
        if (SEG && seg > 0) fetch(a[0], ahead);
        auto operand = [&](int g, uint32_t at) {
            uint32_t from = slot[g] + at;
            if constexpr (SEG) from = __builtin_amdgcn_inverse_ballot_w64(takes[g]) ? from : (uint32_t)plan.lds_zero;
            return *reinterpret_cast<const v4i*>(lds + from);
        };
        constexpr int kAhead = NG > 7 ? 3 : NG < 6 ? NG : 6;       // activation operands in flight
        v4i b[kAhead];
        uint32_t at = ahead.window;
#pragma unroll
        for (int i = 0; i < kAhead; ++i) b[i] = operand(i, at);
        auto step = [&](auto first_c, v4i (&cur)[P], v4i (&nxt)[P], int s) {
            if (s + 1 < s_end) advance(ahead);     // past the end: the last step again
            fetch(nxt, ahead);
            const uint32_t at_next = ahead.window;
            v4i x[NG + kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) x[i] = b[i];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                x[g + kAhead] = g + kAhead < NG ? operand(g + kAhead, at) : operand(g + kAhead - NG, at_next);
#pragma unroll
                for (int q = 0; q < P; ++q)
                    acc[g][q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(cur[q], x[g], decltype(first_c)::value ? v4i{0, 0, 0, 0} : acc[g][q], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < kAhead; ++i) b[i] = x[NG + i];
            at = at_next;
        };
        if (!SEG || seg == 0) step(std::true_type{}, a[0], a[1], s_begin);
        else step(std::false_type{}, a[0], a[1], s_begin);
        int s = s_begin + 1;
        for (; s + 2 <= s_end; s += 2) {
            step(std::false_type{}, a[1], a[0], s);
            step(std::false_type{}, a[0], a[1], s + 1);
        }
        if (s < s_end) step(std::false_type{}, a[1], a[0], s);
    }

    const int oc_first = oc16 * 16 + 4 * quarter;
    auto exists = [&](int g) { return 16 * g + col < plan.part && pix_first + part_at + (uint32_t)(16 * g + col) < npix; };
    const bool full = oc16 * 16 + 16 <= p.OC;
    uint32_t res_word[NG];
    if (OUT == kOutRequant && p.rq.res_i8) {
        if (kStageRes && plan.lds_res) {
#pragma unroll
            for (int g = 0; g < NG; ++g)
                res_word[g] = *reinterpret_cast<const uint32_t*>(lds + plan.lds_res + ((uint32_t)og * tile + part_at + (uint32_t)min(16 * g + col, plan.part - 1)) * 16u + (uint32_t)quarter * 4u);
        } else if (p.rq.res_blocked || p.quad_res) {   // on their way while the sums are put together
            const __amdgpu_buffer_rsrc_t rsrc = word_buffer(p, p.rq.res_i8, p.rq.res_blocked != 0);
            uint32_t off[NG];
            if (full) word_offsets<NG, true>(p, p.rq.res_blocked != 0, oc_first, entry_of, exists, off);
            else word_offsets<NG, false>(p, p.rq.res_blocked != 0, oc_first, entry_of, exists, off);
#pragma unroll
            for (int g = 0; g < NG; ++g) res_word[g] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off[g], 0, 0);
        }
    }
    // digit planes recombined, modulo 2^32
    uint32_t sum[NG][4];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t u = 0;
#pragma unroll
            for (int q = 0; q < P; ++q) u += (uint32_t)acc[g][q][i] << (8 * q);
            sum[g][i] = u;
        }
    auto owner = [&](int g) { return (g << plan.log_wk) / NG; };         // the reduction part that finishes group g
    v4i* const meet = reinterpret_cast<v4i*>(window) + (wave & ((kResidentWaves >> plan.log_wk) - 1)) * (NG * (wk - 1) * 64) + lane;
    if (wk > 1) {                                  // uniform over the workgroup
        __syncthreads();                           // every operand has been read
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (owner(g) != kp)
                meet[(g * (wk - 1) + (kp < owner(g) ? kp : kp - 1)) * 64] = v4i{(int)sum[g][0], (int)sum[g][1], (int)sum[g][2], (int)sum[g][3]};
        __syncthreads();
    }
    auto mine = [&](int g) { return wk == 1 || owner(g) == kp; };        // (true at compile time with one reduction part)
    if (wk > 1) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
            if (mine(g))
                for (int k = 0; k < wk - 1; ++k) {
                    const v4i v = meet[(g * (wk - 1) + k) * 64];
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[g][i] += (uint32_t)v[i];
                }
    }
    const float4 m4 = *reinterpret_cast<const float4*>(s_mult + og * 16 + 4 * quarter), c4 = *reinterpret_cast<const float4*>(s_bias + og * 16 + 4 * quarter);
    const float mult[4] = {m4.x, m4.y, m4.z, m4.w}, bias[4] = {c4.x, c4.y, c4.z, c4.w};
    if (full) finish_tile<OUT, NG, true, SEG>(p, sum, oc_first, mult, bias, res_word, mine, entry_of, exists);
    else finish_tile<OUT, NG, false, SEG>(p, sum, oc_first, mult, bias, res_word, mine, entry_of, exists);
}

// The cut of a call, or false: not for this kernel.
inline bool resident_plan(const SharedParams& p, int planes, int half_tiles, int n_cus, ResidentPlan& plan)
{
    if (p.tKH != 3 || p.tKW != 3 || p.t_stride_h != 1 || p.t_stride_w != 1 || p.t_pad_h != 1 || p.t_pad_w != 1 ||
        p.OH != p.tH || p.OW != p.tW || p.ksplit != 1 || p.masked || planes < 2 || planes > 3)
        return false;
    // (a gate below which the bounds reach, with a scale that turns zero or infinity into NaN: see finish_tile)
    if (p.rq.x_out && p.rq.relu && p.rq.lo < 0.0f && !(p.rq.inv_step > 0.0f && p.rq.inv_step <= 3.0e38f)) return false;
    const ResidentLayer l{(int64_t)p.N * p.OH * p.OW, p.OH, p.OW, p.OC, p.C_pad >> 5, planes, p.n_seg, half_tiles,
                          p.rq.x_out && p.rq.res_i8 && p.rq.res_blocked && ((uintptr_t)p.rq.res_i8 & 15u) == 0};
    if (!resident_plan(l, n_cus, plan)) return false;
    plan.inv_oc_tiles = inverse_of(plan.oc_tiles);
    return true;
}

template <int P, int OUT, int NG, bool SEG>
inline bool launch_resident_one(const SharedParams& p, const ResidentPlan& plan, hipStream_t stream)
{
    auto kernel = k_conv3x3_resident<P, OUT, NG, SEG>;
    static LdsGrant grant;
    if (!grant(kResidentLds, LdsOf{reinterpret_cast<const void*>(kernel)})) return false;
    const unsigned wgs = plan.px_tiles * plan.oc_tiles;
    hipLaunchKernelGGL(kernel, dim3(plan.by_channels ? wgs : (wgs + 7) / 8 * 8), dim3(kResidentWaves * 64), (size_t)plan.lds_bytes, stream, p, plan);
    tl_shared_launch = {kLaunchResident, P, 0, 0, plan.by_channels, NG, 1 << plan.log_wo, 1 << plan.log_wp, 1 << plan.log_wk, plan.part, plan.lds_res > 0};
    return true;
}

// False: not launched, the call goes to the other kernels.
inline bool launch_conv3x3_resident(const SharedParams& p, int planes, int half_tiles, int n_cus, hipStream_t stream)
{
    ResidentPlan plan;
    if (!resident_plan(p, planes, half_tiles, n_cus, plan)) return false;
    auto with_seg = [&](auto p_c, auto out_c, auto ng_c) {
        constexpr int P = decltype(p_c)::value, OUT = decltype(out_c)::value, NG = decltype(ng_c)::value;
        return p.n_seg > 0 ? launch_resident_one<P, OUT, NG, true>(p, plan, stream) : launch_resident_one<P, OUT, NG, false>(p, plan, stream);
    };
    auto with_ng = [&](auto p_c, auto out_c) {
        if (plan.ng == 4) return with_seg(p_c, out_c, std::integral_constant<int, 4>{});
        if (plan.ng == 13) return launch_resident_one<decltype(p_c)::value, decltype(out_c)::value, 13, false>(p, plan, stream);
        return with_seg(p_c, out_c, std::integral_constant<int, 7>{});
    };
    auto with_out = [&](auto p_c) {
        return p.rq.x_out ? with_ng(p_c, std::integral_constant<int, kOutRequant>{}) : with_ng(p_c, std::integral_constant<int, kOutAcc>{});
    };
    return planes == 2 ? with_out(std::integral_constant<int, 2>{}) : with_out(std::integral_constant<int, 3>{});
}

}  // namespace psb
