// Entry points of the integer GEMM / convolution: argument checks and the choice of the
// workgroup tile.  The kernels live in hq_int_gemm_kernel.h.
#include <math.h>

#include <algorithm>

#include "hq_int_gemm_kernel.h"

namespace {

// Tile choice (measured on MI355X; all configurations share one kernel template):
//   - with at least two 64 x 128 tiles per CU, 64-channel tiles at three workgroups per CU win
//     even where 128-channel tiles waste nothing: three waves per SIMD hide the latencies of
//     the chunk loop better than two, which outweighs the extra nibble expansion;
//   - but where those are more than one round (three per CU) and 128 x 128 tiles are not (two per CU), a second, nearly
//     empty round costs as much as the larger tile, which reads fewer operand bytes per product.  us a call, 64 x 128 ->
//     128 x 128: 4096 x 1536 -> 1984 20.6 -> 18.3, 2048 x 2304 -> 3840 26.0 -> 23.3, three weight planes 4096 x 192 -> 1984
//     11.9 -> 11.1.  Not for short K (6200 x 384 -> 1280 13.7 -> 13.85): there the results are most of the time and the third
//     workgroup hides them.  (Of one plane, layers of 576 to 1344 channels that would meet the rule go to hq_linear_fp6.hip.)
//   - otherwise 128 x 128 tiles if there is at least one per CU;
//   - a layer with fewer tiles takes 64 x 64 tiles at four workgroups per CU.
enum class Tile { t128x128, t64x128, t64x64 };

Tile choose_tile(int64_t pixels, int n, int k, int bits, int taps, int64_t cus) {
    if ((bits == 8 ? k : k / 2) % 96 != 0) return Tile::t128x128;
    const int64_t pix128 = (pixels + 127) / 128, tiles64 = pix128 * ((n + 63) / 64), tiles128 = pix128 * ((n + 127) / 128);
    if (bits == 4 && taps <= 3 && taps * k >= 576 && tiles64 > 3 * cus && tiles128 <= 2 * cus) return Tile::t128x128;
    if (n % 64 == 0 && pix128 * (n / 64) >= 2 * cus) return Tile::t64x128;
    return tiles128 >= cus ? Tile::t128x128 : Tile::t64x64;
}

hq_status launch_gemm(const GemmArgs &a, int taps, hq_dtype y_dtype, hipStream_t stream) {
    switch (choose_tile(a.pixels, a.n, a.k, a.bits, taps, hq::compute_units())) {
        case Tile::t128x128: return hq_gemm_launch_128x128(a, taps, y_dtype, stream);
        case Tile::t64x128: return hq_gemm_launch_64x128(a, taps, y_dtype, stream);
        default: return hq_gemm_launch_64x64(a, taps, y_dtype, stream);
    }
}

}  // namespace

// Estimated us of a call: its start, the results (per MB of fp16), and for every 64 input channels (nine taps) what a round of
// a CU's tiles costs plus what each of its tiles costs.  Fitted to 1448 calls of 3x3 layers of 64 to 960 channels, 64 to
// 170000 pixels, rows of 8 to 448: 4 .. 10 % rms.
double hq_tile_us(int64_t pixels, int n, int k, int bits, int sx_static, int had_block) {
    struct Costs {
        double start, result_mb;
        struct { double round, tile; } short_chunks, t64x128, t128x128, t64x64;   // short: K in chunks of 64 codes
    };
    constexpr Costs per_tap{5.6, 0.36, {3.84, 0.38}, {0, 1.18}, {0, 2.90}, {0.90, 0.42}};
    constexpr Costs one_sum{3.7, 0.23, {2.85, 0.98}, {0, 1.26}, {0, 3.10}, {0.90, 0.62}};
    constexpr Costs bytes{5.1, 0.24, {5.67, 1.67}, {0, 2.00}, {0, 4.40}, {1.66, 0.71}};
    constexpr Costs planes{6.4, 0.51, {11.6, 1.31}, {0, 3.44}, {4.00, 7.00}, {3.30, 1.22}};
    const Costs &c = had_block ? planes : bits == 8 ? bytes : sx_static ? one_sum : per_tap;
    const int cus = hq::compute_units();   // (asks the runtime for the device)
    const Tile tile = choose_tile(pixels, n, k, bits, 9, cus);
    const int pt = tile == Tile::t64x64 ? 64 : 128, ct = tile == Tile::t128x128 ? 128 : 64;
    const int per_round = tile == Tile::t64x64 ? 4 : tile == Tile::t64x128 ? 3 : 2;   // (workgroups of a CU)
    const int64_t total = (pixels + pt - 1) / pt * ((n + ct - 1) / ct);
    if (static_cast<double>(total) * ((bits == 8 ? k : k / 2) / 32) * (had_block ? 27 : 9) > 0x7fffffff) return HUGE_VAL;   // (refused)
    const double tiles = static_cast<double>(total) / cus;
    const double rounds = ceil(tiles / per_round), used = (rounds - 1) * per_round + ceil(tiles - (rounds - 1) * per_round);
    const auto &cost = (bits == 8 ? k : k / 2) % 96 != 0 ? c.short_chunks
                       : tile == Tile::t64x128           ? c.t64x128
                       : tile == Tile::t128x128          ? c.t128x128
                                                         : c.t64x64;
    // (groups of 16 channels are stored at once where all are whole, value by value otherwise)
    const double start = c.start + (n % 16 ? 2 : 0), result_mb = c.result_mb + (n % 16 ? 1.2 : 0);
    const double planes_read = had_block && had_block <= 8 ? 2.0 / 3.0 : 1.0;
    return start + static_cast<double>(pixels) * n * 2e-6 * result_mb +
           k / 64 * (cost.round * rounds + cost.tile * used) * planes_read;
}

// The same for linear layers whose K is a multiple of 192: start, results (per MB of fp16; beyond what the caches take they cost more),
// and for every 64 channels of a plane what a round of a CU's tiles and each of its tiles cost.  Fitted to 790 layers of 64 to
// 131072 tokens, 1.5e9 to 6e10 products, one and three planes: 7 % rms.
double hq_tile_linear_us(int64_t pixels, int n, int k, int planes, int cus) {
    const Tile tile = choose_tile(pixels, n, k, 4, planes, cus);
    const int pt = tile == Tile::t64x64 ? 64 : 128, ct = tile == Tile::t128x128 ? 128 : 64;
    const int per_round = tile == Tile::t64x64 ? 4 : tile == Tile::t64x128 ? 3 : 2;   // (workgroups of a CU)
    const double tiles = static_cast<double>((pixels + pt - 1) / pt * ((n + ct - 1) / ct)) / cus;
    const double rounds = ceil(tiles / per_round), used = (rounds - 1) * per_round + ceil(tiles - (rounds - 1) * per_round);
    const double result_mb = static_cast<double>(pixels) * n * 2e-6, steps = k / 64 * planes;
    const double start = 3.46 + result_mb * (n % 16 ? 1.76 : 0.153) + std::max(0.0, result_mb - 64) * 0.015;
    switch (tile) {
        case Tile::t64x128: return start + steps * 0.141 * used;
        case Tile::t128x128: return start + steps * 0.216 * used + 0.89 * rounds;
        default: return start + steps * (0.096 * rounds + 0.048 * used);
    }
}

namespace {

// The kernels index pixels with 32 bits and address the packed operands with
// 32-bit byte offsets; a 3x3 tap shifts an activation offset by up to w + 1 pixels
// before it is clamped, which must not wrap past 2^32 either.
bool fits_32bit(int64_t pixels, int w, int n, int taps, int k) {
    const int64_t lim = 0xFFFFFFFFLL;
    return pixels < 0x7FFFFFFFLL && (pixels + w + 2) * (k / 2) <= lim &&
           static_cast<int64_t>(n) * taps * (k / 2) <= lim;
}

// k_unit: what k must be a multiple of (64 for the kernels that fetch whole 64-code chunks; 8 where the
// kernel for other channel counts can take over)
hq_status check_common(const uint8_t *xq, const float *x_scale, const uint8_t *wq, const float *w_scale,
                       const void *bias, int64_t pixels, int n, int k, const void *y, hq_dtype y_dtype,
                       int k_unit = 64) {
    if (y_dtype != HQ_F16 && y_dtype != HQ_F32 && y_dtype != HQ_I32) return HQ_ERR_DTYPE;
    if (!xq || !wq || !y) return HQ_ERR_NULL;
    if (y_dtype != HQ_I32 && (!x_scale || !w_scale)) return HQ_ERR_NULL;
    if (pixels <= 0 || n <= 0 || k <= 0 || k % k_unit != 0 || k >= 131072) return HQ_ERR_SHAPE;
    if (!hq::aligned16(xq) || !hq::aligned16(wq) || !hq::aligned16(y)) return HQ_ERR_ALIGN;
    if ((reinterpret_cast<uintptr_t>(x_scale) & 3u) || (reinterpret_cast<uintptr_t>(w_scale) & 3u) ||
        (reinterpret_cast<uintptr_t>(bias) & 1u))
        return HQ_ERR_ALIGN;
    return HQ_OK;
}

// One 192-channel slice of 4-bit codes and about one 64 x 64 output tile per CU or fewer: the wave-split kernel, which has no
// activation tile to expand first (1 x 64 x 64 x 192: 8.4 us against 9.2; 1 x 16 x 16 x 192 -> 100: 8.6 against 9.4).  From two
// slices on the resident kernel wins there too (16 x 8 x 8 x 960: 15.4 against 17.8, 23 x 12 x 12 x 384: 13.6 against 16.8).
bool takes_wave_split(int64_t pixels, int c_in, int c_out, int bits) {
    return bits == 4 && c_in == 192 && ((pixels + 63) / 64) * ((c_out + 63) / 64) * 4 <= 5 * hq::compute_units();
}

// Layers of ragged channels that the kernel for few channels finishes sooner: results of 32 bits where groups of eight channels are not
// whole, which the 6-bit kernels store one by one.  us, resident / few channels, 64 x 64 pixels: 8 -> 626 fp32 25 / 19, one int32 sum 23 / 17,
// 24 -> 626 25 / 20 and 23 / 18, 40 -> 626 25 / 23 and 23 / 21, 72 -> 626 27 / 27 and 24 / 25, 8 -> 20 11.0 / 10.7; 8 x 8 pixels 8 -> 59 11.0 / 11.7.
bool few_channels_conv3x3(int64_t pixels, int c_in, int c_out, hq_dtype y_dtype) {
    return c_in % 64 != 0 && y_dtype != HQ_F16 && c_out % 8 != 0 && c_out >= 32 && pixels > 128 && c_in < (y_dtype == HQ_I32 ? 64 : 40);
}
// Linear layers, int32 sums: 30000 x 8 -> 627 94 / 60, 8000 x 120 -> 627 32 / 22, 2000 x 40 -> 201 6.4 / 5.7; for fewer results to a channel the
// products count: 2000 x 200 -> 201 6.7 / 7.4, 500 x 120 -> 41 4.4 / 5.0.
bool few_channels_linear(int64_t m, int k, int n, hq_dtype y_dtype) {
    return k % 64 != 0 && y_dtype == HQ_I32 && n % 8 != 0 && k < 256 && m * n > static_cast<int64_t>(k) * 4340;
}

}  // namespace

namespace {

// bits: 4 (packed pairs of codes) or 8 (int8 codes, one per byte)
hq_status int_linear(const uint8_t *xq, const float *x_scale, const uint8_t *wq, const float *w_scale,
                     const void *bias, int64_t m, int n, int k, void *y, hq_dtype y_dtype, int sx_static,
                     int bits, void *stream) {
    hq_status st = check_common(xq, x_scale, wq, w_scale, bias, m, n, k, y, y_dtype, bits == 4 ? 8 : 64);
    if (st != HQ_OK) return st;
    if (!fits_32bit(m, 1, n, 1, bits == 8 ? 2 * k : k)) return HQ_ERR_UNSUPPORTED;
    GemmArgs a{xq, x_scale, wq, w_scale, bias, y, static_cast<uint32_t>(m), n, k, 1, 1, 0, 0, 0, 1, sx_static,
               1.0f, bits};
    if (bits == 4 && !few_channels_linear(m, k, n, y_dtype)) {
        st = hq_linear_fp6_launch(a, 1, y_dtype, static_cast<hipStream_t>(stream));
        if (st != HQ_ERR_UNSUPPORTED) return st;
    }
    if (k % 64 != 0) return hq_gemm_launch_anyk(a, 1, y_dtype, static_cast<hipStream_t>(stream));
    return launch_gemm(a, 1, y_dtype, static_cast<hipStream_t>(stream));
}

// Linear layer of the Single scheme: the weights are three digit planes, the kernel keeps one
// integer sum per plane and weighs plane p by 16^p when it folds the sums into the fp32 result.
hq_status int_linear_single(const uint8_t *xq, const float *x_scale, const uint8_t *wq3, const float *w_scale,
                            const void *bias, int64_t m, int n, int k, int had_block, void *y, hq_dtype y_dtype,
                            void *stream) {
    hq_status st = check_common(xq, x_scale, wq3, w_scale, bias, m, n, k, y, y_dtype);
    if (st != HQ_OK) return st;
    if (!hq::pow2_upto_128(had_block) || k % had_block != 0) return HQ_ERR_SHAPE;
    if (!fits_32bit(m, 1, n, 3, k)) return HQ_ERR_UNSUPPORTED;
    const float norm = static_cast<float>(1.0 / sqrt(static_cast<double>(had_block)));
    GemmArgs a{xq, x_scale, wq3, w_scale, bias, y, static_cast<uint32_t>(m), n, k, 1, 1, 0, 0, 0, 1, 0, norm, 4};
    // |W_int H_raw| <= 8 x block: up to block 8 that is two signed base-16 digits ([-136, 119]) and the third
    // plane is zero, so its pass is skipped (the integer output keeps all three sums)
    const int planes = had_block <= 8 && y_dtype != HQ_I32 ? 2 : 3;
    st = hq_linear_fp6_launch(a, planes, y_dtype, static_cast<hipStream_t>(stream));
    if (st != HQ_ERR_UNSUPPORTED) return st;
    return launch_gemm(a, planes, y_dtype, static_cast<hipStream_t>(stream));
}

hq_status int_conv2d(const uint8_t *xq, const float *x_scale, const uint8_t *wq, const float *w_scale,
                     const void *bias, int nb, int h, int w, int c_in, int c_out, int r, int s, int stride,
                     int pad, void *y, hq_dtype y_dtype, int sx_static, int bits, void *stream) {
    if (nb <= 0 || h <= 0 || w <= 0 || r <= 0 || s <= 0 || stride <= 0 || pad < 0) {
        if (!xq || !wq || !y) return HQ_ERR_NULL;
        return HQ_ERR_SHAPE;
    }
    const int64_t pixels = static_cast<int64_t>(nb) * h * w;
    hq_status st = check_common(xq, x_scale, wq, w_scale, bias, pixels, c_out, c_in, y, y_dtype,
                                bits == 4 && stride == 1 ? 8 : 64);   // (8-bit codes and stride 2: whole 64-code chunks)
    if (st != HQ_OK) return st;
    const bool down = r == 3 && s == 3 && stride == 2 && pad == 1 && !(bits == 8 && sx_static);   // the downsampling convolution
    if (!down && (r != s || (r != 1 && r != 3) || stride != 1 || pad != (r - 1) / 2)) return HQ_ERR_UNSUPPORTED;
    if (!fits_32bit(pixels, w, c_out, r * s, bits == 8 ? 2 * c_in : c_in)) return HQ_ERR_UNSUPPORTED;
    // one sum over all taps: 256 * (64 per product) * (codes per sum) must stay below 2^31
    if (sx_static && static_cast<int64_t>(c_in) * r * s >= 131072) return HQ_ERR_SHAPE;
    GemmArgs a{xq, x_scale, wq, w_scale, bias, y, static_cast<uint32_t>(pixels), c_out, c_in, h, w, 0, 0, 0, 1,
               sx_static, 1.0f, bits};
    hipStream_t st_ = static_cast<hipStream_t>(stream);
    if (down) {   // output [nb, (h - 1) / 2 + 1, (w - 1) / 2 + 1, c_out]: the tile kernel's stride-2 form
        a.stride = 2;
        a.h_out = (h - 1) / 2 + 1;
        a.w_out = (w - 1) / 2 + 1;
        a.in_pixels = static_cast<uint32_t>(pixels);
        a.pixels = static_cast<uint32_t>(static_cast<int64_t>(nb) * a.h_out * a.w_out);
        return hq_gemm_launch_64x64(a, 9, y_dtype, st_);
    }
    if (r == 3 && !few_channels_conv3x3(pixels, c_in, c_out, y_dtype)) {
        if (takes_wave_split(pixels, c_in, c_out, bits)) return hq_conv3x3_wave_launch(a, y_dtype, st_);
        st = hq_resident_launch(a, 0, y_dtype, st_);
        if (st != HQ_ERR_UNSUPPORTED) return st;
    }
    if (r == 1 && bits == 4 && !few_channels_linear(pixels, c_in, c_out, y_dtype)) {
        st = hq_linear_fp6_launch(a, 1, y_dtype, st_);
        if (st != HQ_ERR_UNSUPPORTED) return st;
    }
    if (c_in % 64 != 0) return hq_gemm_launch_anyk(a, r * s, y_dtype, st_);
    return launch_gemm(a, r * s, y_dtype, st_);
}

// The paper's width-axis convolution: the activations arrive as three digit planes of the integers
// (X~ H_c)_int H_c,raw; the kernel walks 27 steps (plane-major), keeps one integer sum per plane
// over its nine taps (taps outside the image load zeros) and weighs plane p by 16^p.
hq_status int_conv2d_width(const uint8_t *xu3, const float *x_scale, const uint8_t *wq, const float *w_scale,
                           const void *bias, int nb, int h, int w, int c_in, int c_out, int r, int s, int stride,
                           int pad, int had_block, void *y, hq_dtype y_dtype, void *stream) {
    if (nb <= 0 || h <= 0 || w <= 0 || r <= 0 || s <= 0 || stride <= 0 || pad < 0) {
        if (!xu3 || !wq || !y) return HQ_ERR_NULL;
        return HQ_ERR_SHAPE;
    }
    const int64_t pixels = static_cast<int64_t>(nb) * h * w;
    hq_status st = check_common(xu3, x_scale, wq, w_scale, bias, pixels, c_out, c_in, y, y_dtype);
    if (st != HQ_OK) return st;
    if (!hq::pow2_upto_128(had_block) || had_block > 64 || w % had_block != 0) return HQ_ERR_SHAPE;
    if (r != 3 || s != 3 || (stride != 1 && stride != 2) || pad != 1) return HQ_ERR_UNSUPPORTED;
    // three planes of activations behind one 32-bit offset; 256 * 64 * (codes per plane sum) below 2^31
    if (!fits_32bit(3 * pixels, w, c_out, 9, c_in)) return HQ_ERR_UNSUPPORTED;
    if (static_cast<int64_t>(c_in) * 9 >= 131072) return HQ_ERR_SHAPE;
    const float norm = static_cast<float>(1.0 / sqrt(static_cast<double>(had_block)));
    GemmArgs a{xu3, x_scale, wq, w_scale, bias, y, static_cast<uint32_t>(pixels), c_out, c_in, h, w, 0, 0, 0, 1,
               1, norm, 4};
    if (stride == 2) {   // output [nb, (h - 1) / 2 + 1, (w - 1) / 2 + 1, c_out]: the tile kernel's stride-2 form
        a.stride = 2;
        a.h_out = (h - 1) / 2 + 1;
        a.w_out = (w - 1) / 2 + 1;
        a.in_pixels = static_cast<uint32_t>(pixels);
        a.pixels = static_cast<uint32_t>(static_cast<int64_t>(nb) * a.h_out * a.w_out);
        return hq_gemm_launch_64x64(a, had_block <= 8 ? 18 : 27, y_dtype, static_cast<hipStream_t>(stream));
    }
    // The resident kernel adds all products in fp32, weights as 0..15: exact while 15 x (8 x block) x 9 c_in stays within
    // 2^24.  (Its two operand planes hold digits 1 and 2 together up to block 32.)
    if (had_block <= 32 && 15LL * 8 * had_block * 9 * c_in <= 1 << 24) {
        st = hq_resident_launch(a, had_block, y_dtype, static_cast<hipStream_t>(stream));
        if (st != HQ_ERR_UNSUPPORTED) return st;
    }
    // |q H_raw| <= 8 x block: up to block 8 the third digit plane is zero and its nine steps are skipped
    return launch_gemm(a, had_block <= 8 ? 18 : 27, y_dtype, static_cast<hipStream_t>(stream));
}

}  // namespace

extern "C" hq_status hq_int_linear(const uint8_t *xq, const float *x_scale, const uint8_t *wq,
                                   const float *w_scale, const void *bias, int64_t m, int n, int k,
                                   void *y, hq_dtype y_dtype, void *stream) {
    return int_linear(xq, x_scale, wq, w_scale, bias, m, n, k, y, y_dtype, 0, 4, stream);
}

extern "C" hq_status hq_int_linear_static(const uint8_t *xq, const float *x_scale, const uint8_t *wq,
                                          const float *w_scale, const void *bias, int64_t m, int n, int k,
                                          void *y, hq_dtype y_dtype, void *stream) {
    return int_linear(xq, x_scale, wq, w_scale, bias, m, n, k, y, y_dtype, 1, 4, stream);
}

extern "C" hq_status hq_int_conv2d(const uint8_t *xq, const float *x_scale, const uint8_t *wq,
                                   const float *w_scale, const void *bias, int nb, int h, int w, int c_in,
                                   int c_out, int r, int s, int stride, int pad, void *y, hq_dtype y_dtype,
                                   void *stream) {
    return int_conv2d(xq, x_scale, wq, w_scale, bias, nb, h, w, c_in, c_out, r, s, stride, pad, y, y_dtype, 0,
                      4, stream);
}

extern "C" hq_status hq_int_conv2d_static(const uint8_t *xq, const float *x_scale, const uint8_t *wq,
                                          const float *w_scale, const void *bias, int nb, int h, int w,
                                          int c_in, int c_out, int r, int s, int stride, int pad, void *y,
                                          hq_dtype y_dtype, void *stream) {
    return int_conv2d(xq, x_scale, wq, w_scale, bias, nb, h, w, c_in, c_out, r, s, stride, pad, y, y_dtype, 1,
                      4, stream);
}

extern "C" hq_status hq_int_linear_single(const uint8_t *xq, const float *x_scale, const uint8_t *wq3,
                                          const float *w_scale, const void *bias, int64_t m, int n, int k,
                                          int had_block, void *y, hq_dtype y_dtype, void *stream) {
    return int_linear_single(xq, x_scale, wq3, w_scale, bias, m, n, k, had_block, y, y_dtype, stream);
}

extern "C" hq_status hq_int_conv2d_width(const uint8_t *xu3, const float *x_scale, const uint8_t *wq,
                                         const float *w_scale, const void *bias, int nb, int h, int w,
                                         int c_in, int c_out, int r, int s, int stride, int pad,
                                         int had_block, void *y, hq_dtype y_dtype, void *stream) {
    return int_conv2d_width(xu3, x_scale, wq, w_scale, bias, nb, h, w, c_in, c_out, r, s, stride, pad, had_block,
                            y, y_dtype, stream);
}

extern "C" hq_status hq_int_linear_i8(const int8_t *xq, const float *x_scale, const int8_t *wq,
                                      const float *w_scale, const void *bias, int64_t m, int n, int k,
                                      void *y, hq_dtype y_dtype, void *stream) {
    return int_linear(reinterpret_cast<const uint8_t *>(xq), x_scale, reinterpret_cast<const uint8_t *>(wq), w_scale,
                      bias, m, n, k, y, y_dtype, 0, 8, stream);
}

extern "C" hq_status hq_int_conv2d_i8(const int8_t *xq, const float *x_scale, const int8_t *wq,
                                      const float *w_scale, const void *bias, int nb, int h, int w, int c_in,
                                      int c_out, int r, int s, int stride, int pad, void *y, hq_dtype y_dtype,
                                      void *stream) {
    return int_conv2d(reinterpret_cast<const uint8_t *>(xq), x_scale, reinterpret_cast<const uint8_t *>(wq), w_scale,
                      bias, nb, h, w, c_in, c_out, r, s, stride, pad, y, y_dtype, 0, 8, stream);
}

extern "C" const char *hq_int_conv2d_kernel_name(int nb, int h, int w, int c_in, int c_out, int r, int s, int stride,
                                                 int pad, int static_scale, int bits) {
    if (nb <= 0 || h <= 0 || w <= 0 || c_in <= 0 || c_out <= 0 || (bits != 4 && bits != 8)) return "unsupported";
    if (r == 3 && s == 3 && stride == 2 && pad == 1) return c_in % 64 == 0 ? "tile (stride 2)" : "unsupported";
    if (r != s || (r != 1 && r != 3) || stride != 1 || pad != (r - 1) / 2) return "unsupported";
    if (c_in % 8 != 0 || (bits == 8 && c_in % 64 != 0)) return "unsupported";
    if (r == 3) {   // (from here on as in int_conv2d)
        const int64_t pixels = static_cast<int64_t>(nb) * h * w;
        if (takes_wave_split(pixels, c_in, c_out, bits)) return "wave-split";
        if (const char *cut = hq_resident_cut_name(pixels, w, c_in, c_out, bits, static_scale)) return cut;
    }
    if (r == 1 && bits == 4)
        if (const char *cut = hq_linear_cut_name(static_cast<int64_t>(nb) * h * w, c_out, c_in)) return cut;
    return c_in % 64 != 0 ? "small-channel-count" : "tile";
}
