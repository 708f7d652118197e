// NHWC 3x3 convolution of 4-bit codes on the 6-bit floating-point matrix instruction (hq_fp6.h), with
// the activation tile expanded once and resident in LDS.
//
// A workgroup owns XW groups of 128 consecutive pixels and a run of blocks of 32 output channels; a wave's
// result tile is 32 channels x 128 pixels.  The codes of the pixels, and those of W + 1 pixels either side, are fetched
// once, expanded to 6-bit fields and kept in LDS as planes
//     [64-channel step][lane half][row] of 16-byte operand parts, then of 8-byte parts,
// so that a wave's operand read of 32 consecutive rows is two contiguous runs for any row shift: 224 bytes per clock
// and CU measured, against 126 with the halves of a row next to each other.  Weights go from memory straight into
// registers, one unit ahead; there is no barrier between the filling of the tile and the end of a phase.
//
// A unit is one tap and one slice of KS steps: 7 vector instructions per 16 weight codes to expand them (hq_fp6.h),
// KS operand reads and KS MFMAs for each of the four 32-pixel tiles, and (per-pixel scales) one fold of 16
// values into the fp32 sums per tile.  What bounds it: vector issue and matrix pipe together.  A 192-channel unit has
// 5.3 (fold) + 3.5 (weights) + about 1 vector instructions per MFMA; a loop of such a mix alone takes 30 ns per MFMA
// and SIMD (21 ns without them: on random codes the chip holds 1.6 .. 2.1 GHz), the kernel's 31 .. 33 ns.  The other half
// of a launch is what surrounds the loop: start and first loads (2 us), expanding the tile (2 .. 4 us; 24
// instructions per 16 codes for the signed form), exchange and results (2 .. 5 us).
//
// Measured (3x3, 4-bit, us, buffers rotating beyond the last-level cache; before: int8 kernels that expanded nibbles
// at every use or streamed both operands through LDS), per-pixel scales / one scale:
//     16 x 64 x 64 x 192   31.1 -> 27.3 / 28.4 -> 27.1      16 x 8 x 8 x 960            17.8 -> 15.4 / 17.8 -> 15.0
//     16 x 32 x 32 x 384   31.9 -> 25.2 / 30.5 -> 25.1       8 x 16 x 16 x 960          32.6 -> 22.0 / 31.4 -> 21.5
//     16 x 16 x 16 x 576   24.0 -> 20.1 / 26.8 -> 20.2       3 x 45 x 27 x 320 -> 200   32.7 -> 11.1 / 28.8 -> 10.8
//
// Phases.  The tasks (pixel group, channel block) of a workgroup are dealt out to its NW waves in phases: NW at a
// time, then the remainder in powers of two, the units of a task shared by 2, 4 or 8 waves whose sums meet in
// LDS in a fixed order.  So all waves multiply about the same number of units whatever the channel count is.
//
// Digit planes (the width-axis form).  The activations are numbers u = d0 + 16 d1 + 256 d2 in three planes of base-16
// digits; d1 + 16 d2 lies in -16..16 up to transform block 32, which E2M3 still holds, so two operand planes are enough:
// the fill combines the upper two, and their products are multiplied by 16 by the block exponent of the matrix
// instruction.  A unit expands its weights once for both planes.  16 x 16 x 16 x 576, block 16: 33.8 us against 76.7 on the
// tile kernel, which streams weights and all three planes through LDS.
//
// 8-bit codes (the form of 16-byte operands on v_mfma_i32_32x32x32_i8, nothing to expand on either side; the two
// 32-channel halves of a step take the places of two operand planes, each with weights of its own).  Matrix time is twice
// that of 4-bit codes and the fold converts 16 values more per tile; matrix and vector time add up almost fully here as
// there.  us per pass with the quantiser, tile kernel -> this one: 16 x 32 x 32 x 384 51.5 -> 44.1, 16 x 64 x 64 x 192
// 63.7 -> 45.1, 16 x 16 x 16 x 576 44.0 -> 32.1, 16 x 8 x 8 x 960 48.2 -> 22.5, 3 x 45 x 27 x 320 -> 200 51.3 -> 15.9,
// 1 x 8 x 8 x 64 (launch) 26.7 -> 11.2.
//
// Which layers come here and which stay on the tile kernel: choose_kernel in hq_resident.hip.
//
// Weights carry an offset of 8 (hq_fp6.h; not those of 8 bits): a sum exceeds the wanted one by 8 x (sum of the activation
// codes it covers), the same for all channels: a per-pixel correction from a table of code sums.  With one scale all of it
// is exact.
// With per-pixel scales the correction is subtracted at the end from sums in fp32 that hold it, one fold per tap and slice,
// which costs digits: the 2-norm error is 2e-7 .. 3e-7 where code sums are small, up to 1.5e-5 where the codes of a pixel
// have one sign (64 .. 960 channels), below the 2.07e-4 of rounding to fp16 (seen there: nothing in six digits, or 0.2 %).
// fp32 results would lose digits, so their sums start at minus the correction (one fp16 matrix step per tap and tile), run
// over all slices of a tap, and are folded once: 6e-8 for both, as with sums in integers.  That form is slower (us, fp32
// results: 16 x 32 x 32 x 384 28.1 -> 30.7, 16 x 64 x 64 x 192 34.9 -> 39.2) and would cost fp16 results 2 us as well.
#pragma once
#include <type_traits>

#include "hq_fp6.h"
#include "hq_int_gemm_kernel.h"

struct ResidentArgs {
    const uint8_t *xq;   // [pixels, k/2]
    const float *sx;     // [pixels], or one value
    const uint8_t *wq;   // [n, taps, k/2]
    const float *sw;     // [n]
    const void *bias;    // [n] of the output dtype, or null
    void *y;             // [pixels, n]; per-tap integer output [pixels, 9, n], zero-filled before the launch
    uint32_t pixels;
    int n, k, h, w;
    int in_planes;       // kResPlanes: planes that are not all zeros (2 or 3)
    float out_scale;     // times the one scale
    uint32_t w_magic, w_shift, h_magic, h_shift;   // exact division of a pixel index by w and by h
    int slices, chunk;             // K slices of KS steps, and how many are resident at a time
    int xw_log2;                   // pixel groups of 128 per workgroup
    int cb;                        // channel blocks of 32 per workgroup
    uint32_t ch_groups, px_tiles;  // workgroups: channel runs x pixel tiles
    uint32_t d_magic, d_shift;     // exact division of a tile index by the count that runs fastest
    int ch_major;                  // neighbouring workgroups share the channels (else the pixels)
    int rows;                      // rows of the LDS image, odd, the last one all zeros
    int wide;                      // the exchange area has 16 KiB per wave (else 8)
    uint32_t part8, exchange, tables;   // LDS offsets: 8-byte parts, exchange / staging area, tables
};

namespace {

constexpr int kResPerTap = 0;   // 3x3, per-pixel scales: one sum per tap, combined in fp32
constexpr int kResSum = 1;      // 3x3, one scale: one sum over all taps
constexpr int kResPlanes = 2;   // as kResSum, with activations u = d0 + 16 (d1 + 16 d2) in three digit planes, |d1 + 16 d2| <= 16
constexpr int kResBytes = 3;    // as kResPerTap, with 8-bit codes on the int8 instruction

// Barrier that orders LDS only: __syncthreads() would also wait for the wave's global loads (weights requested
// ahead) and stores.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Buffer accesses: uniform base and bound in scalar registers, a 32-bit offset per lane; loads beyond the bound
// return zeros, stores beyond it are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, static_cast<int>(bytes), 0x00027000);
}
__device__ __forceinline__ v4i buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off) {
    return __builtin_bit_cast(
        v4i, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(lane_off), static_cast<int>(uniform_off), 0));
}
__device__ __forceinline__ void buffer_store16(const v4i &v, __amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off) {
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, static_cast<int>(lane_off),
                                           static_cast<int>(uniform_off), 0);
}

__host__ __device__ constexpr int resident_table_bytes(int kind, int px, int rows, int cb) {
    return (kind == kResPerTap || kind == kResBytes ? 9 : 0) * px * 4 + 2 * px * 4 + 2 * rows * 4 + cb * 256;
}

// -sum / 8 in every value of the lane's pixel, that is -8 x the sum of its activation codes in the unit (1/64) of the
// products: a matrix step of K = 8 in fp16 of which one lane half uses two places (sum = lo + 1024 hi; every part and product
// is exact).
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v16f minus_eighth_of(const v4h &weights, int sum) {
    const v4h b = {static_cast<_Float16>(static_cast<short>(sum & 1023)),
                   static_cast<_Float16>(static_cast<short>(sum >> 10)), 0, 0};
    return __builtin_amdgcn_mfma_f32_32x32x8f16(weights, b, v16f{}, 0, 0, 0);
}

template <int OUT, int KIND, int KS>
__global__ __launch_bounds__(512, 2) void resident_kernel(ResidentArgs a) {
    constexpr bool BYTES = KIND == kResBytes, FOLD = KIND == kResPerTap || BYTES, INT_TAPS = OUT == kOutI32 && FOLD;
    constexpr bool WHOLE_TAPS = KIND == kResPerTap && OUT == kOutF32;   // (see the offset of the weights above)
    constexpr int TAPS = 9, NT = 4;
    // planes in memory, operand planes in LDS (BYTES: the two 32-channel halves of a step) and of the weights
    constexpr int IN = KIND == kResPlanes ? 3 : BYTES ? 2 : 1, PL = KIND == kResPlanes || BYTES ? 2 : 1, WP = BYTES ? 2 : 1;
    constexpr int STEP = BYTES ? 64 : 32;   // bytes of a step of 64 codes
    using Out = typename OutT<OUT>::type;
    using Operand = std::conditional_t<BYTES, v4i, v8i>;
    using Acc = std::conditional_t<BYTES, v16i, v16f>;
    constexpr float UNIT = BYTES ? 1.0f : 64.0f;   // a product of two codes is 1 / UNIT in the accumulators
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int tid = threadIdx.x, nt = blockDim.x, nw = nt >> 6;
    const int lane = tid & 63, l = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cb = BYTES ? a.k : a.k >> 1, steps = a.k >> 6, rows = a.rows;
    const int px_wg = 128 << a.xw_log2;
    const int halo = a.w + 1;

    // workgroup b runs on XCD b % 8: every XCD gets a contiguous run of tiles
    const uint32_t nwg = gridDim.x, xcd = blockIdx.x & 7, q8 = nwg >> 3, r8 = nwg & 7;
    const uint32_t tile = xcd * q8 + (xcd < r8 ? xcd : r8) + (blockIdx.x >> 3);
    const uint32_t fast = a.ch_major ? a.px_tiles : a.ch_groups;
    const uint32_t slow_i = hq::div_magic31(tile, fast, a.d_magic, a.d_shift), fast_i = tile - slow_i * fast;
    const uint32_t p0 = (a.ch_major ? fast_i : slow_i) * px_wg;
    const int c_wg = static_cast<int>(a.ch_major ? slow_i : fast_i) * a.cb * 32;
    const int blocks = min(a.cb, (a.n - c_wg + 31) / 32);   // channel blocks of this workgroup

    float *s_sx = reinterpret_cast<float *>(lds + a.tables);
    float *s_corr = s_sx + (FOLD ? TAPS : 0) * px_wg;
    int *s_mask = reinterpret_cast<int *>(s_corr + px_wg);
    float *s_rowscale = reinterpret_cast<float *>(s_mask + px_wg);
    int *s_sum = reinterpret_cast<int *>(s_rowscale + rows);   // code sums [row] of the slices so far
    float *s_sw = reinterpret_cast<float *>(s_sum + rows);
    float *s_bias = s_sw + a.cb * 32;
    short *s_part = reinterpret_cast<short *>(s_bias + a.cb * 32);   // WHOLE_TAPS: code sums [resident slice][row]

    // ---- phases: tasks and shares ---------------------------------------------------------------------------
    // tasks first .. first + (nw >> kl) - 1, each by 1 << kl waves; wave wv has task first + wv >> kl, share wv mod
    int left = blocks << a.xw_log2, first = 0, kl = 0;
    auto shrink = [&]() {
        kl = 0;
        while ((nw >> kl) > left) ++kl;
    };
    shrink();
    int c0 = 0, px_l = 0, u = 0, u_end = 0;   // first channel, first pixel (local), units of this wave's task
    uint32_t w_lane = 0;                      // this lane's weight row
    const int resident0 = a.chunk < a.slices ? a.chunk : a.slices;
    int s0 = 0, s1 = resident0;               // resident slices
    auto begin_task = [&]() {
        const int task = first + (wv >> kl), share = wv & ((1 << kl) - 1);
        px_l = (task & ((1 << a.xw_log2) - 1)) * 128;
        c0 = c_wg + (task >> a.xw_log2) * 32;
        const int co = c0 + tile_row_to_channel(l);
        w_lane = static_cast<uint32_t>(co < a.n ? co : a.n - 1) * (TAPS * cb) + h * 16;
        const int units = TAPS * (s1 - s0);
        u = share * units >> kl;
        u_end = (share + 1) * units >> kl;
    };
    // unit u of the resident slices: tap u / (s1 - s0), slice s0 + u % (s1 - s0)
    v4i raw[WP][KS];   // weights of the next unit as they lie in memory
    const __amdgpu_buffer_rsrc_t w_buf = buffer_of(a.wq, static_cast<uint32_t>(a.n) * (TAPS * cb));
    auto load_weight = [&](int k, int tap, int slice) {
        const int step = slice * KS + k < steps ? slice * KS + k : 0;   // (past the channels: activations are zero)
#pragma unroll
        for (int i = 0; i < WP; ++i)
            raw[i][k] = buffer_load16(w_buf, w_lane, static_cast<uint32_t>(tap * cb + step * STEP + i * 32));
    };
    auto load_weights = [&](int tap, int slice) {
#pragma unroll
        for (int k = 0; k < KS; ++k) load_weight(k, tap, slice);
    };

    // ---- activation tile: packed codes -> signed 6-bit fields ------------------------------------------------
    // Wave items (32 rows, slice): lane = (row, lane half), KS 16-byte pieces each; the code sum of a row's
    // slice is that of two neighbouring lanes.
    const int row_items = (px_wg + 2 * halo + 31) >> 5;
    const uint32_t last = a.pixels - 1;
    const int64_t row_pixel0 = static_cast<int64_t>(p0) - halo;
    const int f_row = lane >> 1, f_half = lane & 1;
    const uint32_t plane_bytes = a.pixels * static_cast<uint32_t>(cb);
    const __amdgpu_buffer_rsrc_t x_buf = buffer_of(a.xq, BYTES ? plane_bytes : IN * plane_bytes);
    auto fill_load = [&](v4i (&p)[IN][KS], int item) {
        const int sl = item / row_items, row = (item - sl * row_items) * 32 + f_row;
        // (rows outside the tensor wrap or lie beyond the bound and read as zeros; they are never used)
        const uint32_t off = (static_cast<uint32_t>(p0) - halo + row) * cb + f_half * 16;
#pragma unroll
        for (int i = 0; i < IN; ++i)
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                p[i][k] = v4i{0, 0, 0, 0};
                if ((s0 + sl) * KS + k < steps && i < a.in_planes)
                    p[i][k] = buffer_load16(x_buf, off, i * (BYTES ? 32u : plane_bytes) + ((s0 + sl) * KS + k) * STEP);
            }
    };
    auto fill_store = [&](const v4i (&p)[IN][KS], int item) {
        const int sl = item / row_items, row = (item - sl * row_items) * 32 + f_row;
        int sum = 0;
        if (row < rows - 1) {
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                if constexpr (BYTES) {
#pragma unroll
                    for (int i = 0; i < PL; ++i)
                        *reinterpret_cast<v4i *>(lds + ((((sl * PL + i) * KS + k) * 2 + f_half) * rows + row) * 16) = p[i][k];
                    continue;
                }
                auto codes = [&](const v4i &v, int s) {
                    return sum_codes8(v.x, sum_codes8(v.y, sum_codes8(v.z, sum_codes8(v.w, s))));
                };
                auto put = [&](int plane, const int (&d)[6]) {
                    const int at = (((sl * PL + plane) * KS + k) * 2 + f_half) * rows + row;
                    *reinterpret_cast<v4i *>(lds + at * 16) = v4i{d[0], d[1], d[2], d[3]};
                    *reinterpret_cast<int2 *>(lds + a.part8 + at * 8) = int2{d[4], d[5]};
                };
                int d[6];
                fp6_signed16(p[0][k].x, p[0][k].y, d[0], d[1], d[2]);
                fp6_signed16(p[0][k].z, p[0][k].w, d[3], d[4], d[5]);
                put(0, d);
                sum = codes(p[0][k], sum);
                if constexpr (KIND == kResPlanes) {
                    fp6_upper16(p[1][k].x, p[2][k].x, p[1][k].y, p[2][k].y, d[0], d[1], d[2]);
                    fp6_upper16(p[1][k].z, p[2][k].z, p[1][k].w, p[2][k].w, d[3], d[4], d[5]);
                    put(1, d);
                    sum += 16 * codes(p[1][k], 0) + 256 * codes(p[2][k], 0);
                }
            }
        }
        if constexpr (!BYTES) {
            sum += __builtin_amdgcn_mov_dpp(sum, 0xB1, 0xF, 0xF, true);   // the other half of the row (lanes 1,0,3,2)
            if (f_half == 0 && row < rows - 1) {
                if constexpr (WHOLE_TAPS) s_part[sl * rows + row] = static_cast<short>(sum);
                else atomicAdd(&s_sum[row], sum);
            }
        }
    };

    // All first loads are requested before any is waited for (a first use costs a trip to HBM).
    v4i p[2][IN][KS];
    begin_task();
    const int first_items = row_items * (s1 - s0);
    fill_load(p[0], wv < first_items ? wv : 0);
    load_weights(u / (s1 - s0), u % (s1 - s0));
    constexpr bool ROW_SCALES = FOLD && !INT_TAPS;
    auto row_scale = [&](int i) {
        int64_t pix = row_pixel0 + i;
        pix = pix < 0 ? 0 : (pix > static_cast<int64_t>(last) ? last : pix);
        return a.sx[pix];
    };
    float t_scale[2] = {}, t_sw = 0.f, t_bias = 0.f;
    if constexpr (ROW_SCALES) {
        t_scale[0] = row_scale(tid);
        t_scale[1] = row_scale(tid + nt);
    }
    if constexpr (OUT != kOutI32) {
        const int c = c_wg + tid < a.n ? c_wg + tid : a.n - 1;
        t_sw = a.sw[c];
        t_bias = a.bias ? to_float(static_cast<const Out *>(a.bias)[c]) : 0.f;
    }
    if constexpr (!WHOLE_TAPS) {
        for (int i = tid; i < rows; i += nt) s_sum[i] = 0;
    }
    for (int i = tid; i < resident0 * PL * KS * 2; i += nt) {   // the row of zeros
        const int at = i * rows + rows - 1;
        *reinterpret_cast<v4i *>(lds + at * 16) = v4i{0, 0, 0, 0};
        if constexpr (!BYTES) *reinterpret_cast<int2 *>(lds + a.part8 + at * 8) = int2{0, 0};
    }
    if constexpr (ROW_SCALES) {
        if (tid < rows) s_rowscale[tid] = t_scale[0];
        if (tid + nt < rows) s_rowscale[tid + nt] = t_scale[1];
        for (int i = tid + 2 * nt; i < rows; i += nt) s_rowscale[i] = row_scale(i);
    }
    if constexpr (OUT != kOutI32) {
        if (tid < blocks * 32) {
            s_sw[tid] = t_sw;
            s_bias[tid] = t_bias;
        }
        for (int i = tid + nt; i < blocks * 32; i += nt) {
            const int c = c_wg + i < a.n ? c_wg + i : a.n - 1;
            s_sw[i] = a.sw[c];
            s_bias[i] = a.bias ? to_float(static_cast<const Out *>(a.bias)[c]) : 0.f;
        }
    }
    lds_barrier();   // the code sums are zero before they are added to

    v16f sum[NT] = {};   // the accumulators themselves, or (FOLD) fp32 combinations of per-tap sums
    for (;;) {           // chunks of resident slices
        const int items = row_items * (s1 - s0);
        for (int item = wv; item < items; item += 2 * nw) {
            if (item + nw < items) fill_load(p[1], item + nw);
            fill_store(p[0], item);
            if (item + nw < items) {
                if (item + 2 * nw < items) fill_load(p[0], item + 2 * nw);
                fill_store(p[1], item + nw);
            }
        }
        lds_barrier();
        // tables of the pixels: tap masks, scales under the taps, corrections
        for (int i = tid; i < px_wg; i += nt) {
            const uint32_t pix = p0 + i;
            const uint32_t q = hq::div_magic31(pix, a.w, a.w_magic, a.w_shift);
            const int ow = static_cast<int>(pix - q * a.w);
            const int oh = static_cast<int>(q - hq::div_magic31(q, a.h, a.h_magic, a.h_shift) * a.h);
            const int cm = (ow > 0 ? 1 : 0) | 2 | (ow + 1 < a.w ? 4 : 0);
            int mask = (oh > 0 ? cm : 0) | (cm << 3) | (oh + 1 < a.h ? cm << 6 : 0);
            if (pix >= a.pixels) mask = 0;
            s_mask[i] = mask;
            float corr = 0.f;
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int row = halo + i + (t / 3 - 1) * a.w + (t % 3 - 1);
                const bool in = (mask >> t) & 1;
                if constexpr (FOLD && !INT_TAPS) {
                    const float s = in ? s_rowscale[row] : 0.f;
                    s_sx[t * px_wg + i] = s;
                    if constexpr (!BYTES && !WHOLE_TAPS) corr = fmaf(s * (8.0f / UNIT), static_cast<float>(s_sum[row]), corr);
                } else if (!BYTES && in) {
                    corr += 8.0f * static_cast<float>(s_sum[row]);
                }
            }
            if constexpr (!WHOLE_TAPS) s_corr[i] = corr;   // (of all slices once the last chunk is resident)
        }
        if constexpr (WHOLE_TAPS) {   // code sums of a slice -> of all resident slices up to it
            for (int i = tid; i < px_wg + 2 * halo; i += nt) {
                int of = s_part[i];
                for (int sl = 1; sl < s1 - s0; ++sl) {
                    of += s_part[sl * rows + i];
                    s_part[sl * rows + i] = static_cast<short>(of);
                }
            }
        }
        lds_barrier();

        for (;;) {   // phases
            int mask[NT];   // kResSum / INT_TAPS: taps inside the image, for the pixels of the four tiles
            if constexpr (!FOLD || INT_TAPS) {
#pragma unroll
                for (int t = 0; t < NT; ++t) mask[t] = s_mask[px_l + t * 32 + l];
            }
            const int lane_row = px_l + l + halo;
            const int ns = s1 - s0;
            int tap = u / ns, sl = u - tap * ns;
            // LDS offsets of this lane's row of tile 0 in the two parts of a unit's first plane; the other tiles and
            // steps lie at fixed distances
            const int plane16 = rows * 32, plane8 = rows * 16;   // from step to step
            struct Base { int b16, b8; };
            auto base_of = [&](int tap, int sl) {
                const int shift = (tap / 3 - 1) * a.w + tap % 3 - 1;
                const int at = (sl * PL * KS * 2 + h) * rows + lane_row;
                return Base{(at + shift) * 16, static_cast<int>(a.part8) + (at + shift) * 8};
            };
            auto load_tile = [&](Operand (&b)[KS], const Base &base, int tap, int t, int plane) {
                int b16 = base.b16 + plane * KS * plane16, b8 = base.b8 + plane * KS * plane8, imm = t;
                if constexpr (!FOLD) {   // taps outside the image read the row of zeros
                    const int row = lane_row + (tap / 3 - 1) * a.w + tap % 3 - 1;
                    const int to = (mask[t] >> tap) & 1 ? t * 32 : rows - 1 - row;
                    b16 += to * 16;
                    b8 += to * 8;
                    imm = 0;
                }
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const v4i lo = *reinterpret_cast<const v4i *>(lds + (b16 + k * plane16) + imm * 512);
                    if constexpr (BYTES) {
                        b[k] = lo;
                    } else {
                        const int2 hi = *reinterpret_cast<const int2 *>(lds + (b8 + k * plane8) + imm * 256);
                        b[k] = v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, 0, 0};
                    }
                }
            };
            // While the MFMAs of tile t run, tile t + 1 is on its way from LDS and the sums of tile t - 1 are folded (of
            // WHOLE_TAPS only where the unit ends the slices of its tap); the next unit's weights are requested as soon as
            // this unit's are expanded.
            Base base = base_of(tap, sl);
            Operand wop[WP][KS], b[2][KS];
            load_tile(b[0], base, tap, 0, 0);
            Acc tap_acc[WHOLE_TAPS ? NT : 1];
            const v4h minus = h ? v4h{} : v4h{-0.125f16, -128.0f16, 0, 0};
            auto codes_upto = [&](int tap, int sl, int t) {
                return static_cast<int>(s_part[sl * rows + lane_row + (tap / 3 - 1) * a.w + tap % 3 - 1 + t * 32]);
            };
            if constexpr (WHOLE_TAPS) {   // the sums of a tap start with the offset of the slices that this wave will add
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    tap_acc[t] = minus_eighth_of(minus, codes_upto(tap, min(ns, sl + u_end - u) - 1, t) -
                                                            (sl ? codes_upto(tap, sl - 1, t) : 0));
            }
            for (; u < u_end; ++u) {
                int tap1 = tap, sl1 = sl;   // the next unit (the last one's operands are requested twice)
                if (u + 1 < u_end) {
                    if (++sl1 == ns) { sl1 = 0; ++tap1; }
                }
                const Base base1 = base_of(tap1, sl1);
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    if constexpr (BYTES) {
#pragma unroll
                        for (int i = 0; i < WP; ++i) wop[i][k] = raw[i][k];
                    } else {
                        int d[6];
                        fp6_offset16(raw[0][k].x, raw[0][k].y, d[0], d[1], d[2]);
                        fp6_offset16(raw[0][k].z, raw[0][k].w, d[3], d[4], d[5]);
                        wop[0][k] = v8i{d[0], d[1], d[2], d[3], d[4], d[5], 0, 0};
                    }
                }
                load_weights(tap1, s0 + sl1);
                Acc unit_acc[WHOLE_TAPS ? 1 : 2];
                auto acc_of = [&](int t) -> Acc & {
                    if constexpr (WHOLE_TAPS) return tap_acc[t];
                    else return unit_acc[t & 1];
                };
                const bool ends = !WHOLE_TAPS || u + 1 == u_end || tap1 != tap;
                float scale[NT];
                int codes[NT] = {};   // WHOLE_TAPS: of the next tap
                if (FOLD && !INT_TAPS && ends) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        scale[t] = s_sx[tap * px_wg + px_l + t * 32 + l];
                        if constexpr (WHOLE_TAPS) codes[t] = codes_upto(tap1, max(min(ns, u_end - u - 1), 1) - 1, t);
                    }
                }
                auto fold = [&](int t) {
                    if constexpr (INT_TAPS) {
                        const uint32_t pix = p0 + px_l + t * 32 + l;
                        if ((mask[t] >> tap) & 1) {
                            const int row = lane_row + (tap / 3 - 1) * a.w + tap % 3 - 1 + t * 32;
                            const int extra = !BYTES && sl == 0 ? 8 * s_sum[row] : 0;
                            int *dst = static_cast<int *>(a.y) + (static_cast<uint64_t>(pix) * 9 + tap) * a.n;
#pragma unroll
                            for (int i = 0; i < 16; ++i) {
                                const int c = c0 + 16 * h + i;
                                if (c < a.n)
                                    atomicAdd(dst + c,
                                              static_cast<int>(acc_of(t)[i] * static_cast<decltype(acc_of(t)[i] + 0)>(UNIT)) - extra);
                            }
                        }
                    } else if constexpr (FOLD) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) sum[t][i] = fmaf(scale[t], static_cast<float>(acc_of(t)[i]), sum[t][i]);
                        if constexpr (WHOLE_TAPS) tap_acc[t] = minus_eighth_of(minus, codes[t]);
                    }
                };
#pragma unroll
                for (int t = 0; t < NT; ++t) {
#pragma unroll
                    for (int plane = 0; plane < PL; ++plane) {
                        const int now = t * PL + plane, next = now + 1;
                        if (next < NT * PL) load_tile(b[next & 1], base, tap, next / PL, next % PL);
                        else load_tile(b[0], base1, tap1, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if constexpr (BYTES) {
                            Acc c = plane ? acc_of(t) : Acc{};
#pragma unroll
                            for (int k = 0; k < KS; ++k)
                                c = __builtin_amdgcn_mfma_i32_32x32x32_i8(wop[plane][k], b[now & 1][k], c, 0, 0, 0);
                            acc_of(t) = c;
                        } else {
                            v16f c = WHOLE_TAPS ? acc_of(t) : FOLD ? v16f{} : sum[t];
#pragma unroll
                            for (int k = 0; k < KS; ++k)
                                c = plane ? mfma_fp6_times16(wop[0][k], b[now & 1][k], c) : mfma_fp6(wop[0][k], b[now & 1][k], c);
                            if constexpr (FOLD) acc_of(t) = c;
                            else sum[t] = c;
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if (t > 0 && plane == 0 && ends) fold(t - 1);
                    }
                }
                if (ends) fold(NT - 1);
                tap = tap1;
                sl = sl1;
                base = base1;
            }
            if (s1 < a.slices) break;   // the sums go on with the next chunk (one phase: host)

            // ---- results of the phase --------------------------------------------------------------------------
            if constexpr (!INT_TAPS) {
                // Tasks shared by 2, 4 or 8 waves: in every round a wave hands half of what it holds to a partner and
                // adds the partner's sums of the other half, until it holds 4 >> kl pixel tiles (or half a tile).
                int tile0 = 0, half0 = 0;   // what it holds: tiles tile0 .., or half half0 of tile tile0
                v4i *const outbox = reinterpret_cast<v4i *>(lds + a.exchange) + wv * 512 + lane;
                auto exchange = [&](auto KEEP, int distance) {   // KEEP: values per lane that stay
                    constexpr int keep = decltype(KEEP)::value;
                    const int upper = wv & distance ? 1 : 0;
                    const v4i *const inbox = reinterpret_cast<const v4i *>(lds + a.exchange) + (wv ^ distance) * 512 + lane;
                    lds_barrier();   // the area is free (it may lie over the activation tile)
#pragma unroll
                    for (int i = 0; i < keep; i += 4) {
                        v4i out;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int at = i + e, other = keep + i + e;
                            const float lo = sum[at >> 4][at & 15], hi = sum[other >> 4][other & 15];
                            out[e] = __float_as_int(upper ? lo : hi);
                            sum[at >> 4][at & 15] = upper ? hi : lo;
                        }
                        outbox[i * 16] = out;
                    }
                    lds_barrier();
#pragma unroll
                    for (int i = 0; i < keep; i += 4) {
                        const v4i in = inbox[i * 16];
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[(i + e) >> 4][(i + e) & 15] += __int_as_float(in[e]);
                    }
                    return upper;
                };
                if (kl >= 2 && a.wide) {
                    // room for everything: every wave writes all its sums and adds up its own 64 >> kl values of all waves
                    const int kws = 1 << kl, share = wv & (kws - 1);
                    v4i *const box = reinterpret_cast<v4i *>(lds + a.exchange) + lane;
                    lds_barrier();
#pragma unroll
                    for (int i = 0; i < 64; i += 4)
                        box[(wv * 16 + i / 4) * 64] =
                            v4i{__float_as_int(sum[i >> 4][i & 15]), __float_as_int(sum[i >> 4][(i + 1) & 15]),
                                __float_as_int(sum[i >> 4][(i + 2) & 15]), __float_as_int(sum[i >> 4][(i + 3) & 15])};
                    lds_barrier();
                    sum[0] = v16f{};
                    for (int j = 0; j < kws; ++j) {
                        const v4i *const from = box + ((wv - share + j) * 16 + (share * 16 >> kl)) * 64;
#pragma unroll
                        for (int i = 0; i < 16; i += 4) {
                            if (i == 8 && kl == 3) break;
                            const v4i in = from[i * 16];
#pragma unroll
                            for (int e = 0; e < 4; ++e) sum[0][i + e] += __int_as_float(in[e]);
                        }
                    }
                    tile0 = share * 4 >> kl;
                    half0 = kl == 3 ? share & 1 : 0;
                    lds_barrier();   // (the results go through the area)
                } else {
                    if (kl >= 1) tile0 = 2 * exchange(std::integral_constant<int, 32>{}, 1 << (kl - 1));
                    if (kl >= 2) tile0 += exchange(std::integral_constant<int, 16>{}, 1 << (kl - 2));
                    if (kl >= 3) half0 = exchange(std::integral_constant<int, 8>{}, 1);
                }

                const float one_scale = !FOLD && OUT != kOutI32 ? a.sx[0] * a.out_scale : 1.0f;
                // results of eight sums v of a pixel with correction corr, channels ct .. ct + 7 (in the workgroup)
                auto scaled = [&](const float (&v)[8], float corr, const float *sw, const float *bias, Out (&res)[8]) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if constexpr (OUT == kOutI32) {
                            res[i] = static_cast<int>(v[i] * 64.0f - corr);
                        } else {
                            // (scales of up to the largest float: they are not multiplied by the unit before their codes)
                            const float r = FOLD ? (v[i] - corr) * UNIT : (v[i] * 64.0f - corr) * one_scale;
                            const float y = fmaf(r, sw[i], bias[i]);
                            if constexpr (OUT == kOutF16) res[i] = __float2half_rn(y);
                            else res[i] = y;
                        }
                    }
                };
                const uint32_t rows_left = min(a.pixels - p0, static_cast<uint32_t>(px_wg));
                Out *const y_wg = static_cast<Out *>(a.y) + static_cast<uint64_t>(p0) * a.n;
                const __amdgpu_buffer_rsrc_t y_buf = buffer_of(y_wg, rows_left * static_cast<uint32_t>(a.n * sizeof(Out)));
                const bool vec = a.n % 8 == 0;   // groups of eight channels are whole and 16-byte aligned
                auto store8 = [&](const Out (&res)[8], int px, int c) {
                    if (vec) {
                        // (beyond the bound: dropped)
                        const uint32_t off = c < a.n ? static_cast<uint32_t>(px * a.n + c) * sizeof(Out) : 0x80000000u;
                        buffer_store16(reinterpret_cast<const v4i *>(res)[0], y_buf, off, 0);
                        if constexpr (sizeof(Out) == 4) buffer_store16(reinterpret_cast<const v4i *>(res)[1], y_buf, off + 16, 0);
                    } else if (px < static_cast<int>(rows_left)) {
                        for (int i = 0; i < 8; ++i)
                            if (c + i < a.n) y_wg[static_cast<uint64_t>(px) * a.n + c + i] = res[i];
                    }
                };
                const int ct = c0 - c_wg + 16 * h;
                if (kl < 3) {
                    // fp16: through LDS, [pixel][four 16-byte pieces] of 2 KiB per tile, so that four neighbouring lanes
                    // store the 64 contiguous bytes of a pixel instead of every lane a piece of its own (after an
                    // exchange in the area of the last partner, which nobody else reads)
                    uint8_t *const stage = lds + a.exchange + (kl ? wv ^ 1 : wv) * 8192;
                    float sw[16], bias[16], corr[NT];
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        sw[i] = OUT != kOutI32 ? s_sw[ct + i] : 0.f;
                        bias[i] = OUT != kOutI32 ? s_bias[ct + i] : 0.f;
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const int px = px_l + ((tile0 + t) & (NT - 1)) * 32 + l;
                        corr[t] = WHOLE_TAPS ? 0.f : s_corr[px];
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if (t >= NT >> kl) break;
                        const int px = px_l + (tile0 + t) * 32;
                        Out res[2][8];
#pragma unroll
                        for (int half = 0; half < 2; ++half) {
                            float v[8];
#pragma unroll
                            for (int i = 0; i < 8; ++i) v[i] = sum[t][8 * half + i];
                            scaled(v, corr[t], sw + 8 * half, bias + 8 * half, res[half]);
                        }
                        if constexpr (OUT == kOutF16) {
#pragma unroll
                            for (int half = 0; half < 2; ++half)
                                *reinterpret_cast<v4i *>(stage + t * 2048 + l * 64 + (((2 * h + half) ^ ((l >> 2) & 3)) * 16)) =
                                    *reinterpret_cast<const v4i *>(res[half]);
                        } else {
                            store8(res[0], px + l, c0 + 16 * h);
                            store8(res[1], px + l, c0 + 16 * h + 8);
                        }
                    }
                    if constexpr (OUT == kOutF16) {
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        const int q = lane >> 2, piece = lane & 3;
                        const uint8_t *const from = stage + q * 64 + ((piece ^ ((q >> 2) & 3)) * 16);
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            if (t >= NT >> kl) break;
#pragma unroll
                            for (int half = 0; half < 2; ++half) {
                                Out out[8];
                                *reinterpret_cast<v4i *>(out) = *reinterpret_cast<const v4i *>(from + t * 2048 + half * 1024);
                                store8(out, px_l + (tile0 + t) * 32 + 16 * half + q, c0 + 8 * piece);
                            }
                        }
                    }
                } else {
                    const int px = px_l + tile0 * 32 + l;
                    float v[8], sw[8], bias[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        v[i] = sum[0][i];
                        sw[i] = OUT != kOutI32 ? s_sw[ct + 8 * half0 + i] : 0.f;
                        bias[i] = OUT != kOutI32 ? s_bias[ct + 8 * half0 + i] : 0.f;
                    }
                    Out res[8];
                    scaled(v, WHOLE_TAPS ? 0.f : s_corr[px], sw, bias, res);
                    store8(res, px, c0 + 16 * h + 8 * half0);
                }
            }
            first += nw >> kl;
            left -= nw >> kl;
            if (left == 0) return;
            shrink();
            begin_task();
            load_weights(u / ns, s0 + u % ns);
#pragma unroll
            for (int t = 0; t < NT; ++t) sum[t] = v16f{};
        }

        // ---- next chunk -----------------------------------------------------------------------------------------
        s0 = s1;
        s1 = s0 + a.chunk < a.slices ? s0 + a.chunk : a.slices;
        begin_task();
        fill_load(p[0], wv < row_items * (s1 - s0) ? wv : 0);
        load_weights(u / (s1 - s0), s0 + u % (s1 - s0));
        lds_barrier();   // every wave is done with the resident slices
        if constexpr (INT_TAPS) {   // per-tap sums are corrected with the code sums of their own slices
            for (int i = tid; i < rows; i += nt) s_sum[i] = 0;
            lds_barrier();
        }
    }
}

}  // namespace

// One form's kernels by output type and steps per slice (a file each, so that they compile in parallel).
#define HQ_RESIDENT_FORM(NAME, KIND)                                                                            \
    const void *NAME(int out, int ks) {                                                                         \
        static const void *const kernels[3][3] = {                                                              \
            HQ_RESIDENT_FORM_OUT(kOutF16, KIND), HQ_RESIDENT_FORM_OUT(kOutF32, KIND), HQ_RESIDENT_FORM_OUT(kOutI32, KIND)}; \
        return kernels[out == kOutF16 ? 0 : out == kOutF32 ? 1 : 2][ks - 1];                                    \
    }
#define HQ_RESIDENT_FORM_OUT(OUT, KIND)                                                                         \
    {reinterpret_cast<const void *>(resident_kernel<OUT, KIND, 1>), reinterpret_cast<const void *>(resident_kernel<OUT, KIND, 2>), \
     reinterpret_cast<const void *>(resident_kernel<OUT, KIND, 3>)}
