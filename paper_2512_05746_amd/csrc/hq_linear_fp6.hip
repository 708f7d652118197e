// Linear layers (and 1x1 convolutions) of 4-bit codes on the 6-bit floating-point matrix instruction (hq_fp6.h).
//
// A workgroup owns 32 NT tokens and one block of 32 output channels for each of its 4 or 8 waves.  The tokens' codes are fetched
// and expanded once into LDS (planes [step of 64 channels][lane half][row] of 16- and of 8-byte operand parts) and read by
// all waves; a wave's weights go from memory straight into registers, KS steps ahead, and are expanded beside the products of the
// step before; no barrier between the filling and the results.  Both operands carry an offset of 8, which makes the expansion
// 7 instructions for 16 codes:
//     sum (x + 8)(w + 8) = sum x w + 8 (sum x + 8 K) + 8 sum w;
// the code sums are taken with dot products on the way, and one small fp16 matrix step per tile subtracts them, exactly.
//
// K that is no multiple of 64 (but of 8): the last step is filled up with activation codes of zero, on the way into LDS; what the
// weights' loads find beyond the end of a row then does not matter, since the correction counts it as well.
//
// Digit planes of the weights (the Single scheme: [n, 3, k/2], planes weighing 1, 16, 256): one such product for every plane, folded
// into fp32 sums, the tokens expanded once for all.
//
// What bounds it (2048 x 960 -> 3840, 13.0 us back to back, the int8 tile kernel 14.4): launch and first loads 2.3 us, the
// expansion of the tokens 1.3 (issue of vector instructions), products 4.5 (2.8 of matrix instructions, the rest the expansion
// of the weights beside them), results 1.6 (15.7 MB), from launch to launch 2.  Tiles of 128 tokens halve the weights' loads
// and expansions against 64 (14.1 us with 64); they keep to 128 registers, so that two workgroups of 8 waves share a CU where
// their tokens leave room (up to K = 640).
#include <limits.h>
#include <math.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "hq_buffer.h"
#include "hq_fp6.h"
#include "hq_int_gemm_kernel.h"

namespace {

struct LinearArgs {
    const uint8_t *xq;   // [pixels, k/2]
    const float *sx;     // [pixels], or one value
    const uint8_t *wq;   // [n, planes in memory, k/2]
    const float *sw;     // [n]
    const void *bias;    // [n] of the output dtype, or null
    void *y;             // [pixels, n]
    uint32_t pixels;
    int n, k, sx_static, planes;   // planes multiplied
    float out_scale;               // times the channel scales
    uint32_t row_bytes;            // of a channel's weights, all planes
    int units;                     // of KS steps, the last one padded with activations of zero
    uint32_t ch_groups, px_tiles, d_magic, d_shift;   // workgroups, and exact division by the count that runs fastest
    int ch_major;                  // neighbouring workgroups share the channels (else the tokens)
};

__host__ __device__ constexpr int operand_bytes(int px, int steps) { return steps * 2 * px * 24; }
__host__ __device__ constexpr int table_bytes(int px, int nw) { return px * 8 + nw * (2048 + 256); }

typedef _Float16 v4h __attribute__((ext_vector_type(4)));
__device__ __forceinline__ _Float16 half_of(int v) { return static_cast<_Float16>(static_cast<short>(v)); }

template <int OUT, int NT, int KS, bool PLANES>
__global__ __launch_bounds__(512, !PLANES || NT == 1 ? 4 : NT == 2 ? 3 : 2) void linear_kernel(LinearArgs a) {
    constexpr int PX = 32 * NT, STEP16 = 2 * PX * 16, STEP8 = 2 * PX * 8, AHEAD = 8;
    using Out = typename OutT<OUT>::type;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6;
    const int lane = tid & 63, l = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cb = a.k >> 1, whole = a.k >> 6, steps = (a.k + 63) >> 6, steps_p = a.units * KS;
    const int part8 = steps_p * STEP16;
    int *s_sum = reinterpret_cast<int *>(lds + operand_bytes(PX, steps_p));
    float *s_sx = reinterpret_cast<float *>(s_sum + PX);
    uint8_t *const stages = reinterpret_cast<uint8_t *>(s_sx + PX), *const stage = stages + wv * 2048;
    float *s_sw = reinterpret_cast<float *>(stages + nw * 2048);
    float *s_bias = s_sw + nw * 32;

    // workgroup b runs on XCD b % 8: every XCD gets a contiguous run of tiles
    const uint32_t nwg = gridDim.x, xcd = blockIdx.x & 7, q8 = nwg >> 3, r8 = nwg & 7;
    const uint32_t tile = xcd * q8 + (xcd < r8 ? xcd : r8) + (blockIdx.x >> 3);
    const uint32_t fast = a.ch_major ? a.px_tiles : a.ch_groups;
    const uint32_t slow_i = hq::div_magic31(tile, fast, a.d_magic, a.d_shift), fast_i = tile - slow_i * fast;
    const uint32_t p0 = (a.ch_major ? fast_i : slow_i) * PX;
    const int c_wg = static_cast<int>(a.ch_major ? slow_i : fast_i) * nw * 32, c0 = c_wg + wv * 32;

    // ---- first loads ------------------------------------------------------------------------------------------
    // A wave fills 32 of the tokens at every nw / NT-th step: lane = (row, lane half), one 16-byte piece.
    const int f_half = lane & 1, f_row = wv % NT * 32 + (lane >> 1), f_step0 = wv / NT, f_stride = nw / NT;
    const __amdgpu_buffer_rsrc_t x_buf = buffer_of(a.xq, a.pixels * static_cast<uint32_t>(cb));
    const uint32_t f_lane = (p0 + f_row) * cb + f_half * 16;   // (beyond the tensor: zeros, not used)
    v4i p[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (f_step0 + i * f_stride < whole) p[i] = buffer_load16(x_buf, f_lane, (f_step0 + i * f_stride) * 32);
    const bool f_tail = whole < steps && (whole & (f_stride - 1)) == f_step0;   // the last step is not whole, and this wave's
    v4i p_tail = {0, 0, 0, 0};
    if (f_tail) p_tail = buffer_load16(x_buf, f_lane, whole * 32);
    float t_sx = 0.f, t_sw = 0.f, t_bias = 0.f;
    if constexpr (OUT != kOutI32) {
        if (tid < PX) t_sx = a.sx[a.sx_static ? 0 : p0 + tid < a.pixels ? p0 + tid : a.pixels - 1];
        if (tid < nw * 32) {
            const int c = c_wg + tid < a.n ? c_wg + tid : a.n - 1;
            t_sw = a.sw[c];
            if (a.bias) t_bias = to_float(static_cast<const Out *>(a.bias)[c]);
        }
    }
    const int co = c0 + tile_row_to_channel(l);
    const uint32_t w_lane = static_cast<uint32_t>(co < a.n ? co : a.n - 1) * a.row_bytes + h * 16, w_bytes = static_cast<uint32_t>(a.n) * a.row_bytes;
    const __amdgpu_buffer_rsrc_t w_buf = buffer_of(a.wq, w_bytes);
    uint32_t w_at = 0;   // of the next weights to load, in the row
    // The steps that pad the last unit, and what follows the last plane, read zeros, from the end of the tensor on: the uniform offset
    // is what the bound that the lanes' offsets are held against is less by, so it must not exceed the size.
    const int pad = steps_p - steps;
    auto load_weights = [&](v4i &raw, int k, bool last_unit) {
        raw = buffer_load16(w_buf, w_lane, last_unit && k >= KS - pad ? w_bytes : min(w_at, w_bytes));
        w_at += 32;
    };
    v4i raw[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) load_weights(raw[k], k, a.units == 1);
    if (tid < PX) s_sum[tid] = 0;
    for (int i = tid; i < (steps_p - steps) * 2 * PX; i += nt) {   // padding steps
        const int at = steps * 2 * PX + i;
        *reinterpret_cast<v4i *>(lds + at * 16) = v4i{0, 0, 0, 0};
        *reinterpret_cast<v2i *>(lds + part8 + at * 8) = v2i{0, 0};
    }
    lds_barrier();   // the code sums are zero before they are added to

    // ---- tokens: packed codes -> 6-bit fields ------------------------------------------------------------------
    const Fp6Masks masks;
    int f_sum = 0;
    auto fill_store = [&](const v4i &p, int step) {
        const int at = (step * 2 + f_half) * PX + f_row;
        int d[6];
        fp6_offset16(masks, p.x, p.y, d[0], d[1], d[2]);
        fp6_offset16(masks, p.z, p.w, d[3], d[4], d[5]);
        *reinterpret_cast<v4i *>(lds + at * 16) = v4i{d[0], d[1], d[2], d[3]};
        *reinterpret_cast<v2i *>(lds + part8 + at * 8) = v2i{d[4], d[5]};
        f_sum = sum_codes8(p.x, sum_codes8(p.y, sum_codes8(p.z, sum_codes8(p.w, f_sum))));
    };
    for (int step = f_step0; step < whole; step += AHEAD * f_stride) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            if (step + i * f_stride >= whole) break;
            fill_store(p[i], step + i * f_stride);
            if (step + (i + AHEAD) * f_stride < whole) p[i] = buffer_load16(x_buf, f_lane, (step + (i + AHEAD) * f_stride) * 32);
        }
    }
    if (f_tail) {   // the rest are codes of zero (not in the loop: a branch there waits for the weights too, 256 x 256 -> 256 4.1 -> 4.3 us)
#pragma unroll
        for (int e = 0; e < 4; ++e) p_tail[e] = f_half * 4 + e < (a.k & 63) >> 3 ? p_tail[e] : 0;
        fill_store(p_tail, whole);
    }
    atomicAdd(&s_sum[f_row], f_sum);
    if constexpr (OUT != kOutI32) {
        if (tid < PX) s_sx[tid] = t_sx;
        if (tid < nw * 32) {
            s_sw[tid] = t_sw * a.out_scale;
            s_bias[tid] = t_bias;
        }
    }
    lds_barrier();
    if (c0 >= a.n) return;

    // ---- products ----------------------------------------------------------------------------------------------
    // While the MFMA of a tile runs, the next tile is on its way from LDS and the next step's weights are expanded; KS steps of
    // weights are on their way from memory.
    const int b16_0 = static_cast<int>(lds_address(lds)) + (h * PX + l) * 16;
    const int b8_0 = static_cast<int>(lds_address(lds)) + part8 + (h * PX + l) * 8;
    auto load_tile = [&](v8i &b, int unit, int k, int t) {
        const v4i lo = lds_v4i(b16_0 + unit * (KS * STEP16), k * STEP16 + t * 512);
        const v2i hi = lds_v2i(b8_0 + unit * (KS * STEP8), k * STEP8 + t * 256);
        b = v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, 0, 0};
    };
    // the correction: -(S + sum w) / 8 with S = sum x + 8 K: four places of a matrix step of K = 8 (lo + 1024 hi; the lane halves
    // hold the sums of their halves of the weights; every part and product is exact)
    v16f acc[NT], total[PLANES ? NT : 1];
    if constexpr (PLANES) {
#pragma unroll
        for (int t = 0; t < NT; ++t) total[t] = v16f{};
    }
    float weight = 64.0f;   // of the plane, in units of the accumulators
    int d[6], w_sum = 0;
    auto expand = [&](const v4i &w, int half) {
        if (half == 0) fp6_offset16(masks, w.x, w.y, d[0], d[1], d[2]);
        else fp6_offset16(masks, w.z, w.w, d[3], d[4], d[5]);
    };
    expand(raw[0], 0);
    expand(raw[0], 1);
    auto add_codes = [](const v4i &w, int sum) { return sum_codes8(w.x, sum_codes8(w.y, sum_codes8(w.z, sum_codes8(w.w, sum)))); };
    int w_first = add_codes(raw[0], 0);   // of the coming unit's first step
    // (a unit's first step is expanded, and its place loaded again, with the last step of the unit before)
    int planes_left = PLANES ? a.planes : 1;   // to load
    auto load_first = [&](int unit) {
        if (unit == 0) w_at = --planes_left == 0 ? w_bytes : w_at - pad * 32;   // (the next plane follows the real steps)
        load_weights(raw[0], 0, false);
    };
    load_first(a.units == 1 ? 0 : 1);
    for (int plane = 0; plane < (PLANES ? a.planes : 1); ++plane) {
        w_sum = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = v16f{};
        v8i b[2];
        load_tile(b[0], 0, 0, 0);
        for (int u = 0; u < a.units; ++u) {
            w_sum += w_first;
            const int u1 = u + 1 < a.units ? u + 1 : 0;
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const v8i w = v8i{d[0], d[1], d[2], d[3], d[4], d[5], 0, 0};
                v4i &next = raw[(k + 1) % KS];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    v8i &now = b[(k * NT + t) & 1], &then = b[(k * NT + t + 1) & 1];
                    if (t + 1 < NT) load_tile(then, u, k, t + 1);
                    else if (k + 1 < KS) load_tile(then, u, k + 1, 0);
                    else load_tile(then, u1, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    acc[t] = mfma_fp6(w, now, acc[t]);
                    if (t == 0) expand(next, 0);
                    if (t == (NT > 1)) {
                        expand(next, 1);
                        const int sum = add_codes(next, k + 1 < KS ? w_sum : 0);
                        if (k + 1 < KS) {
                            w_sum = sum;
                            load_weights(next, k + 1, u1 == a.units - 1);
                        } else {
                            w_first = sum;
                            load_first(u1 + 1 < a.units ? u1 + 1 : 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if constexpr (KS * NT % 2) b[0] = b[1];
        }
        const v4h w_part = {half_of(w_sum & 1023), half_of(w_sum >> 10), 1.0f16, 1024.0f16};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int s_x = s_sum[t * 32 + l] + 8 * 64 * steps;
            const _Float16 of_x = h ? 0.0f16 : -0.125f16;
            const v4h x_part = {-0.125f16, -128.0f16, half_of(s_x & 1023) * of_x, half_of(s_x >> 10) * of_x};
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x8f16(w_part, x_part, acc[t], 0, 0, 0);
        }
        if constexpr (PLANES) {
            // (the token's scale comes last: times 256 it would overflow for scales from 1.3e36 on)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) total[t][i] = fmaf(weight, acc[t][i], total[t][i]);
            weight *= 16.0f;
        }
    }

    // ---- results -----------------------------------------------------------------------------------------------
    const uint32_t rows_left = min(a.pixels - p0, static_cast<uint32_t>(PX));
    Out *const y_wg = static_cast<Out *>(a.y) + static_cast<uint64_t>(p0) * a.n;
    const __amdgpu_buffer_rsrc_t y_buf = buffer_of(y_wg, rows_left * static_cast<uint32_t>(a.n * sizeof(Out)));
    const bool vec = a.n % 8 == 0;   // groups of eight channels are whole and 16-byte aligned
    auto store8 = [&](const Out (&res)[8], int px, int c) {
        if (vec) {
            const uint32_t off = c < a.n ? static_cast<uint32_t>(px * a.n + c) * sizeof(Out) : 0x80000000u;   // (beyond the bound: dropped)
            buffer_store16(reinterpret_cast<const v4i *>(res)[0], y_buf, off, 0);
            if constexpr (sizeof(Out) == 4) buffer_store16(reinterpret_cast<const v4i *>(res)[1], y_buf, off + 16, 0);
        } else if (px < static_cast<int>(rows_left)) {
            for (int i = 0; i < 8; ++i)
                if (c + i < a.n) y_wg[static_cast<uint64_t>(px) * a.n + c + i] = res[i];
        }
    };
    float sw[16], bias[16];
    if constexpr (OUT != kOutI32) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            sw[i] = s_sw[wv * 32 + 16 * h + i];
            bias[i] = s_bias[wv * 32 + 16 * h + i];
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float sx = OUT == kOutI32 ? 0.f : s_sx[t * 32 + l];
        Out res[2][8];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float v;
            if constexpr (PLANES) v = total[t][i];
            else v = acc[t][i] * 64.0f;
            if constexpr (OUT == kOutI32) res[i >> 3][i & 7] = static_cast<int>(v);
            else {
                const float y = fmaf(sx * v, sw[i], bias[i]);
                if constexpr (OUT == kOutF16) res[i >> 3][i & 7] = __float2half_rn(y);
                else res[i >> 3][i & 7] = y;
            }
        }
        if constexpr (OUT == kOutF16) {   // through LDS, so that four neighbouring lanes store the 64 contiguous bytes of a token
#pragma unroll
            for (int half = 0; half < 2; ++half)
                *reinterpret_cast<v4i *>(stage + l * 64 + (((2 * h + half) ^ ((l >> 2) & 3)) * 16)) =
                    *reinterpret_cast<const v4i *>(res[half]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int q = lane >> 2, piece = lane & 3;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                Out out[8];
                const uint8_t *from = stage + half * 1024 + q * 64 + (piece ^ ((q >> 2) & 3)) * 16;
                *reinterpret_cast<v4i *>(out) = *reinterpret_cast<const v4i *>(from);
                store8(out, t * 32 + 16 * half + q, c0 + 8 * piece);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            store8(res[0], t * 32 + l, c0 + 16 * h);
            store8(res[1], t * 32 + l, c0 + 16 * h + 8);
        }
    }
}

constexpr int kUnits[3][4] = {{8, 5, 4, 3}, {4, 3, 2, 2}, {4, 3, 2, 2}};   // KS of the tiles of 32, 64 and 128 tokens

template <int OUT, bool PLANES, int NT>
const void *kernel_of(int i) {
    constexpr const int *ks = kUnits[NT >> 1];
    switch (i) {
        case 0: return reinterpret_cast<const void *>(linear_kernel<OUT, NT, ks[0], PLANES>);
        case 1: return reinterpret_cast<const void *>(linear_kernel<OUT, NT, ks[1], PLANES>);
        case 2: return reinterpret_cast<const void *>(linear_kernel<OUT, NT, ks[2], PLANES>);
        default: return reinterpret_cast<const void *>(linear_kernel<OUT, NT, ks[3], PLANES>);
    }
}

template <int OUT, bool PLANES>
const void *kernel_of(int nt_log2, int i) {
    return nt_log2 == 0 ? kernel_of<OUT, PLANES, 1>(i) : nt_log2 == 1 ? kernel_of<OUT, PLANES, 2>(i) : kernel_of<OUT, PLANES, 4>(i);
}

struct Cut {
    int nt_log2, unit, nw, lds;   // unit: of kUnits
    bool ok;
};

// Steps of a unit: the longest way ahead that costs at most 1/8 of padding, else the least padding.
int choose_unit(int steps, int nt_log2) {
    int best = 0, best_pad = INT_MAX;
    for (int i = 0; i < 4; ++i) {
        const int ks = kUnits[nt_log2][i], pad = (steps + ks - 1) / ks * ks - steps;
        if (pad <= steps / 8) return i;
        if (pad < best_pad) { best = i; best_pad = pad; }
    }
    return best;
}

Cut lay_out(int k, int nt_log2, int nw) {
    Cut c{nt_log2, choose_unit((k + 63) / 64, nt_log2), nw, 0, false};
    const int ks = kUnits[nt_log2][c.unit], px = 32 << nt_log2;
    c.lds = operand_bytes(px, ((k + 63) / 64 + ks - 1) / ks * ks) + table_bytes(px, nw);
    c.ok = c.lds <= kLdsPerCu;
    return c;
}

// Estimated us of a cut: start, results (per MB of fp16), rounds of workgroups (each with the latency of its steps), and for
// every CU the expansion of tokens, the expansion of weights, the products and the tiles stored.  Fitted to 222 calls of 1 to
// 131072 tokens, 64 to 4096 channels in, 8 to 5120 out, six cuts each: 12 % rms; the cut it picks is 0.8 % off the best one
// on average.
double cut_us(const Cut &c, int pixels, int n, int k, int planes, int cus) {
    const int nt = 1 << c.nt_log2, blocks = (n + 31) / 32, steps = (k + 63) / 64;
    const int ks = kUnits[c.nt_log2][c.unit], steps_p = (steps + ks - 1) / ks * ks;
    const int64_t wgs = static_cast<int64_t>((pixels + 32u * nt - 1) >> (5 + c.nt_log2)) * ((blocks + c.nw - 1) / c.nw);
    const double per_cu = ceil(static_cast<double>(wgs) / cus);
    const int waves = planes == 1 || nt == 1 ? 16 : nt == 2 ? 12 : 8;   // (of a CU, by registers)
    const int resident = std::max(1, std::min(kLdsPerCu / c.lds, waves / c.nw));
    const double rounds = ceil(per_cu / resident);
    const int active = std::min(c.nw, blocks);
    return 2.22 + 0.103 * 2e-6 * static_cast<double>(pixels) * n + rounds * (1.03 + 0.0983 * steps_p * planes) +
           per_cu * (0.0286 * steps * nt + (0.0025 * nt + 0.009) * steps_p * active * planes + 0.037 * active * nt);
}

// Whether this kernel takes the layer, and its cut.  The tile kernel is at its best where K is a multiple of 192 (its stages
// are 96 bytes of K; other K go by stages of 32) and n one of 16 (it stores groups of 16 channels whole, others value by value).
// Where both are so it keeps the layers below 1.5e9 products (1024 x 960 -> 960: 5.5 against 6.1 us) and from 1536 channels on,
// where the tile of 128 tokens leaves room for four waves only (2924 x 1536 -> 1968: 19.3 against 15.8).  Below 32 channels out one
// wave of four has work (30454 x 1152 -> 24: 8.8 / 7.1).  Of the rest, layers of 192 and 384 channels of one plane come here (8192 x 384 ->
// 1152 11.4 / 12.0; 105 of 111 are faster by 3 % and more, one is 20 % slower); from 576 on, and for digit planes, the two estimates
// decide, which are 10 and 7 % off, so it has to be 8 % ahead for small layers and not 5 % behind for large ones (77907 x 1344 -> 64
// 25.8 / 14.8, 23950 x 960 -> 544 26.7 / 19.9, 44867 x 768 -> 576 40.8 / 30.9; 2048 x 960 -> 3840 13.0 / 14.4, 57956 x 1344 -> 296 44.4 / 81.7).
// K that are no multiple of 64 go to the kernel of hq_int_gemm_anyk.hip only below one step and 2^20 products (27 x 40 -> 24 4.0 / 4.5;
// 2209 x 24 -> 88 6.1 / 4.2, 4096 x 200 -> 400 11.2 / 5.1, 8192 x 920 -> 1152 120 / 20; 200 random layers 0.66 of the time), for many tokens
// and one group of eight channels out, of which the waves for the others have nothing to do (30000 x 40 -> 6 4.7 / 5.9, 30000 x 200 -> 6
// 6.2 / 6.7; 8000 x 40 -> 6 4.6 / 4.8), and where 32 tokens do not fit the LDS.
// For other K this kernel is up to 2.5 times faster (64 x 640 -> 640: 4.7 against 7.2 us, 8192 x 640 -> 640: 9.0 against 10.7,
// 512 x 4096 -> 1024: 14 against 30), save for many rounds of tiles of 32 tokens (9535 x 4096 -> 1920: 188 against 107 of the tile
// kernel; K of 4088 does not go there, 852 us on the kernel of hq_int_gemm_anyk.hip, so the rule is for multiples of 64 only: 213 here).
Cut choose_cut(int pixels, int n, int k, int planes) {
    Cut best{};
    if (n >= 1 << 21) return best;   // (a tile's results lie within 2 GiB of their first)
    const double products = static_cast<double>(pixels) * n * k * planes;
    const bool tile_k = k % 192 == 0;
    if (k % 64 && ((k < 64 && products < 1 << 20) || (n <= 8 && pixels > 16384 && k < 256))) return best;
    if (tile_k && (n < 32 || (n % 16 == 0 && products < 1.5e9) || !lay_out(k, 2, 8).ok)) return best;
    const int cus = hq::compute_units();   // (asks the runtime for the device: once)
    double best_us = HUGE_VAL;
    for (int nt_log2 = 0; nt_log2 < 3; ++nt_log2)
        for (int nw = 4; nw <= 8; nw += 4) {
            const Cut c = lay_out(k, nt_log2, nw);
            const double us = c.ok ? cut_us(c, pixels, n, k, planes, cus) : HUGE_VAL;
            if (us < best_us) { best = c; best_us = us; }
        }
    if (k % 64 == 0 && best.ok && best.nt_log2 == 0 && !lay_out(k, 1, 4).ok) {
        const int64_t wgs = static_cast<int64_t>((pixels + 31u) / 32) * (((n + 31) / 32 + best.nw - 1) / best.nw);
        best.ok = wgs <= 2 * cus;
    }
    if (tile_k && (k >= 576 || planes > 1) && best.ok) {
        const double us = best_us + (n % 8 ? 0.95 * 2e-6 * static_cast<double>(pixels) * n : 0);   // (stored value by value)
        best.ok = hq_tile_linear_us(pixels, n, k, planes, cus) >= (products < 3e9 || k < 384 ? 1.08 : 0.95) * us;
    }
    return best;
}

}  // namespace

// For the diagnostic: nullptr if the layer is one for the tile kernel.
const char *hq_linear_cut_name(int64_t pixels, int n, int k) {
    if (pixels >= INT_MAX) return nullptr;   // (refused)
    const Cut c = choose_cut(static_cast<int>(pixels), n, k, 1);
    if (!c.ok) return nullptr;
#define HQ_LINEAR_NAMES(TOKENS, KS) \
    {"linear (" TOKENS " tokens, 4 waves, units of " KS ")", "linear (" TOKENS " tokens, 8 waves, units of " KS ")"}
    static const char *const names[3][4][2] = {   // [tokens][kUnits][waves]
        {HQ_LINEAR_NAMES("32", "8"), HQ_LINEAR_NAMES("32", "5"), HQ_LINEAR_NAMES("32", "4"), HQ_LINEAR_NAMES("32", "3")},
        {HQ_LINEAR_NAMES("64", "4"), HQ_LINEAR_NAMES("64", "3"), HQ_LINEAR_NAMES("64", "2"), HQ_LINEAR_NAMES("64", "2")},
        {HQ_LINEAR_NAMES("128", "4"), HQ_LINEAR_NAMES("128", "3"), HQ_LINEAR_NAMES("128", "2"), HQ_LINEAR_NAMES("128", "2")}};
#undef HQ_LINEAR_NAMES
    return names[c.nt_log2][c.unit][c.nw == 8];
}

// HQ_ERR_UNSUPPORTED, with nothing launched: the layer is one for the tile kernel.
hq_status hq_linear_fp6_launch(const GemmArgs &g, int planes, hq_dtype y_dtype, hipStream_t stream) {
    if (planes > 1 && y_dtype == HQ_I32) return HQ_ERR_UNSUPPORTED;
    const Cut c = choose_cut(static_cast<int>(g.pixels), g.n, g.k, planes);
    if (!c.ok) return HQ_ERR_UNSUPPORTED;
    const hq::LaunchCheck check;   // samples the thread's error state before anything is launched
    LinearArgs a{};
    a.xq = g.xq; a.sx = g.sx; a.wq = g.wq; a.sw = g.sw; a.bias = g.bias; a.y = g.y;
    a.pixels = g.pixels; a.n = g.n; a.k = g.k; a.sx_static = g.sx_static; a.planes = planes; a.out_scale = g.out_scale;
    a.row_bytes = static_cast<uint32_t>(g.k / 2) * (planes > 1 ? 3 : 1);
    const int ks = kUnits[c.nt_log2][c.unit];
    a.units = ((g.k + 63) / 64 + ks - 1) / ks;
    const int px = 32 << c.nt_log2;
    const int64_t px_tiles = (static_cast<int64_t>(g.pixels) + px - 1) / px, ch_groups = ((g.n + 31) / 32 + c.nw - 1) / c.nw;
    if (px_tiles * ch_groups > 0x7fffffff) return HQ_ERR_UNSUPPORTED;
    a.px_tiles = static_cast<uint32_t>(px_tiles);
    a.ch_groups = static_cast<uint32_t>(ch_groups);
    // the larger operand is the one that an XCD's run of tiles shares
    a.ch_major = static_cast<int64_t>(g.n) * (planes > 1 ? 3 : 1) > static_cast<int64_t>(g.pixels);
    const hq::Magic31 md = hq::magic31(a.ch_major ? a.px_tiles : a.ch_groups);
    a.d_magic = md.m; a.d_shift = md.s;
    const void *fn;
    int out;
    if (planes > 1) {
        out = y_dtype == HQ_F16 ? 3 : 4;
        fn = y_dtype == HQ_F16 ? kernel_of<kOutF16, true>(c.nt_log2, c.unit) : kernel_of<kOutF32, true>(c.nt_log2, c.unit);
    } else {
        out = y_dtype == HQ_F16 ? 0 : y_dtype == HQ_F32 ? 1 : 2;
        fn = out == 0 ? kernel_of<kOutF16, false>(c.nt_log2, c.unit) : out == 1 ? kernel_of<kOutF32, false>(c.nt_log2, c.unit)
                                                                             : kernel_of<kOutI32, false>(c.nt_log2, c.unit);
    }
    static std::atomic<uint64_t> allowed[5][3][4];
    const hq_status st = allow_lds(fn, allowed[out][c.nt_log2][c.unit]);
    if (st != HQ_OK) return st;
    void *args[] = {&a};
    if (hipLaunchKernel(fn, dim3(static_cast<unsigned>(px_tiles * ch_groups)), dim3(64 * c.nw), args, c.lds, stream) != hipSuccess)
        return HQ_ERR_LAUNCH;
    return check.status();
}
