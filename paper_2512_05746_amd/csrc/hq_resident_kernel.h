// NHWC 3x3 convolution of 4-bit codes on the 6-bit floating-point matrix instruction (hq_fp6.h), with
// the activation tile expanded once and resident in LDS.
//
// A workgroup owns XW groups of 128 consecutive pixels and a run of blocks of 32 output channels; a wave's
// result tile is 32 channels x 128 pixels.  The codes of the pixels, and those of W + 1 pixels either side, are fetched
// once, expanded to 6-bit fields and kept in LDS as planes
//     [64-channel step][lane half][row] of 16-byte operand parts, then of 8-byte parts,
// so that a wave's operand read of 32 consecutive rows is two contiguous runs for any row shift (4 clocks a KiB, without
// conflicts).  Weights pass through a ring in LDS of the wave's own; there is no barrier between the filling of the tile and the
// end of a phase.
//
// A step is 64 channels of one tap: 14 vector instructions to expand the weights (hq_fp6.h), one operand read and one MFMA for
// each of the four 32-pixel tiles; per-pixel scales: one fold of 16 values a tile into the fp32 sums for every tap.  What bounds
// it: such MFMAs alone take 33 clocks (a loop of them holds 1.4 GHz, the short one here 1.9 .. 2.1), with the operand reads 34 (two
// waves a SIMD), with ring and direct-to-LDS loads 48, with 4 vector instructions each 51, and every 2 scalar instructions
// an MFMA cost 8 more: a wave issues in order, and what it issues beside an MFMA adds to it.  So steps come in groups of three (below):
// slots of the ring, places of the expanded weights and distances in LDS are constants, requests advance the lane's offset on the
// way; 38 instructions a step instead of 62.  us a call, a step at a time -> groups of three, and the start's arguments loaded at
// once: per-pixel scales 16 x 32 x 32 x 384 25.1 -> 23.6, 8 x 16 x 16 x 960 21.6 -> 20.3; one scale 24.9 -> 23.3; 8 bits 34.0 -> 32.7;
// over 1200 random layers 0.92 .. 0.945 of the time, none more than 2.4 % slower.
// The other half of a launch is what surrounds the loop: start and first loads (2 us: instructions of two waves a SIMD, 7 clocks
// each, and 100 KiB of requests), expanding the tile (2 .. 4 us; 24 instructions per 16 codes for the signed form), exchange and
// results (2 .. 5 us).
//
// Before the steps came in groups (3x3, 4-bit, us a call, weights in L2; weights in registers for every form -> through the ring):
//     per-pixel scales: 8 x 16 x 16 x 960 23.4 -> 21.9, 3 x 45 x 27 x 320 -> 200 11.4 -> 10.8, 3 x 44 x 44 x 576 -> 152 13.3 -> 13.1
//     one scale:       16 x 32 x 32 x 384 26.2 -> 25.1, 4 x 46 x 46 x 960 -> 488 63.4 -> 60.3
//
// Phases.  The tasks (pixel group, channel block) of a workgroup are dealt out to its NW waves in phases: NW at a
// time, then the remainder in powers of two, the units of a task shared by 2, 4 or 8 waves whose sums meet in
// LDS in a fixed order.  So all waves multiply about the same number of units whatever the channel count is.
//
// Digit planes (the width-axis form).  The activations are numbers u = d0 + 16 d1 + 256 d2 in three planes of base-16
// digits; d1 + 16 d2 lies in -16..16 up to transform block 32, which E2M3 still holds, so two operand planes are enough:
// the fill combines the upper two, and their products are multiplied by 16 by the block exponent of the matrix
// instruction.  A unit expands its weights once for both planes.  16 x 16 x 16 x 576, block 16: 28.9 us against 76.7 on the
// tile kernel, which streams weights and all three planes through LDS.
//
// 8-bit codes (the form of 16-byte operands on v_mfma_i32_32x32x32_i8, nothing to expand on either side; the two
// 32-channel halves of a step take the places of two operand planes, each with weights of its own).  Matrix time is twice
// that of 4-bit codes and bounds it: 42 clocks an MFMA of 32, at the 1.5 GHz that the chip holds under them.  us a call,
// weights in registers and a fold of twice the instructions for every 192 channels -> this form, before the steps came in groups:
// 16 x 32 x 32 x 384 40.3 -> 34.4, 2 x 24 x 40 x 640 25.9 -> 20.1.
//
// One scale: taps outside the image must add nothing.  Their products are multiplied by 2^-127 (the block exponent that the matrix
// instruction takes for every column) instead of reading a row of zeros, which would cost every tile an address of its own
// in every step; what they leave, below 1e-35, is rounded away before the sums are scaled.
//
// Channel counts that are no multiple of 64 (but of 8): the last step of a tap is filled up with activation codes of zero, whatever
// the weights' loads find beyond the tap.  us a call, the kernel of hq_int_gemm_anyk.hip -> this one: 2 x 32 x 32 x 200 31.7 -> 9.4,
// 4 x 32 x 32 x 328 50.6 -> 14.0.  It keeps layers that it writes sooner (few_channels_conv3x3 in hq_int_gemm.hip) and the integer sums of taps.
//
// Which layers come here and which stay on the tile kernel: choose_kernel in hq_resident.hip.
//
// Weights carry an offset of 8 (hq_fp6.h; not those of 8 bits): a sum exceeds the wanted one by 8 x (sum of the activation
// codes it covers), the same for all channels: a per-pixel correction from a table of code sums.  With one scale all of it
// is exact.
// With per-pixel scales the fp32 sums start from minus the correction and then hold it in part, which costs digits: the 2-norm
// error is 2e-7 .. 3e-7 where code sums are small, up to 1.5e-5 where the codes of a pixel have one sign (64 .. 960 channels),
// below the 2.07e-4 of rounding to fp16 (seen there: nothing in six digits, or 0.2 %).  fp32 results would lose digits, so there
// the sums of a tap start at minus its correction (one fp16 matrix step per tap and tile): 6e-8, as with sums in integers.  So do
// they for fp16 results of channel counts that are no multiple of 64: 0.02 % of these differ from the exact result rounded once, as
// with sums in integers, against 0.1 .. 0.4 % (8 to 952 channels).
#pragma once
#include <stddef.h>

#include <type_traits>

#include "hq_buffer.h"
#include "hq_fp6.h"
#include "hq_int_gemm_kernel.h"

struct ResidentArgs {
    // What the start of a workgroup needs, 32 words that it loads together.
    const uint8_t *xq;   // [pixels, k/2]
    const uint8_t *wq;   // [n, taps, k/2]
    const float *sx;     // [pixels], or one value
    const float *sw;     // [n]
    const void *bias;    // [n] of the output dtype, or null
    uint32_t pixels;
    int n, k, w;
    int chunk;                     // steps of 64 channels that are resident at a time
    int xw_log2;                   // pixel groups of 128 per workgroup
    int cb;                        // channel blocks of 32 per workgroup
    int waves;                     // 4 or 8
    uint32_t tiles, fast;          // workgroups: channel runs x pixel tiles; those of the kind that runs fastest
    uint32_t d_magic, d_shift;     // exact division of a tile index by that count
    int ch_major;                  // neighbouring workgroups share the channels (else the pixels)
    int rows;                      // rows of the LDS image and one more, odd
    uint32_t part8, ring, tables;  // LDS offsets: 8-byte parts, rings, tables
    uint32_t ring_stride;          // LDS from wave to wave's ring
    uint32_t inverses, inverses_last;   // inverse_of the resident steps and, in the upper half, of their threes; of the last chunk's
    int in_planes;       // kResPlanes: planes that are not all zeros (2 or 3)
    int ring_shared;     // the rings lie in the exchange area
    // The rest.
    void *y;             // [pixels, n]; per-tap integer output [pixels, 9, n], zero-filled before the launch
    int h;
    float out_scale;     // times the one scale
    uint32_t w_magic, w_shift, h_magic, h_shift;   // exact division of a pixel index by w and by h
    int wide;            // the exchange area has 16 KiB per wave (else 8)
    uint32_t exchange;   // LDS offset of the exchange / staging area
};
static_assert(offsetof(ResidentArgs, y) == 128, "32 words");

namespace {

constexpr int kResPerTap = 0;   // 3x3, per-pixel scales: one sum per tap, combined in fp32
constexpr int kResSum = 1;      // 3x3, one scale: one sum over all taps
constexpr int kResPlanes = 2;   // as kResSum, with activations u = d0 + 16 (d1 + 16 d2) in three digit planes, |d1 + 16 d2| <= 16
constexpr int kResBytes = 3;    // as kResPerTap, with 8-bit codes on the int8 instruction
constexpr int kResWholeTaps = 4;   // as kResPerTap, with sums of taps that start at minus their correction (fp32 results; fp16 ones of ragged channels)

// Direct-to-LDS load of 16 bytes a lane: lane i's land at lds_base + 16 i.  Inline assembly, because the compiler cannot tell which
// slot of a ring such a load fills and would wait for all of them before every LDS read; the waits (wait_vmem) are placed by
// hand.  (Its own counted waits stay right: they only wait for more.  m0 is reserved, the compiler sets it before each use of its own
// and takes no clobber of it.)  The lane's offset goes on by `step` first, which takes the place of the wait state after m0.
__device__ __forceinline__ v4i buffer_words(const void *p, uint32_t bytes) {   // a buffer as four scalar registers
    const uint64_t at = reinterpret_cast<uint64_t>(p);
    return v4i{static_cast<int>(at), static_cast<int>(at >> 32 & 0xFFFF), static_cast<int>(bytes), 0x00027000};
}
template <int STEP>
__device__ __forceinline__ void load_to_ring(const v4i &r, uint32_t &lane_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\tv_add_u32_e32 %0, %3, %0\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds"
                 : "+v"(lane_off)
                 : "s"(lds_base), "s"(r), "n"(STEP)
                 : "memory");
}
// Steps of a tap that a form is built for (0: any number).  Not for the integer sums of taps, which their stores bound.  Four steps only
// for sums of codes (us a call, steps in a loop -> unrolled: per-pixel scales 12 x 33 x 33 x 256 16.3 -> 14.5, one scale
// 2 x 30 x 25 x 256 -> 504 10.2 -> 9.4; the width axis, whose operand planes take twice the registers, 2 x 12 x 40 x 256 11.6 -> 12.2).
__host__ __device__ constexpr int resident_unrolled(int kind, int out, int ns) {
    const bool int_taps = out == kOutI32 && (kind == kResPerTap || kind == kResBytes);
    return ns <= (kind == kResPlanes || kind == kResBytes ? 3 : 4) && !int_taps ? ns : 0;
}
// bytes of a step's weights for 32 channels, a slot of a ring
__host__ __device__ constexpr int resident_slot_bytes(int kind) { return kind == kResBytes ? 2048 : 1024; }

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

// x / d rounded down, of inv = 2^15 / d + 1: exact for x d below 2^15
__host__ __device__ constexpr uint32_t inverse_of(int d) { return 32768u / static_cast<uint32_t>(d) + 1; }
__device__ __forceinline__ int quotient(int x, uint32_t inv) { return static_cast<int>(static_cast<uint32_t>(x) * inv >> 15); }

// The arguments, and the index of the thread, read anew: what a part of the kernel derives from them is computed there instead of
// being held (and, for want of registers, spilled) over the loop of matrix instructions.  A load of scalars takes 300 clocks, so the
// start has its own loaded at once (one after the other as they are needed they cost 0.6 us).
typedef const __attribute__((address_space(4))) ResidentArgs KernelArgs;
__device__ __forceinline__ KernelArgs &args_again() {
    uint64_t at = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr());
    asm volatile("" : "+s"(at));
    return *reinterpret_cast<KernelArgs *>(at);
}
__device__ __forceinline__ void start_args(ResidentArgs &a) {
    typedef int v16w __attribute__((ext_vector_type(16)));
    typedef const __attribute__((address_space(4))) v16w KernelWords;
    const uint64_t at = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr());
    v16w words[2] = {reinterpret_cast<KernelWords *>(at)[0], reinterpret_cast<KernelWords *>(at)[1]};
    asm volatile("" : "+s"(words[0]), "+s"(words[1]));
    __builtin_memcpy(&a, words, sizeof words);
}
__device__ __forceinline__ int thread_again() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// RING: slots of the ring in LDS through which weights pass, 3 or, where there is less room, 2; 0: straight from memory.
// NS: 0, or the steps of a tap that are resident at a time, 1 .. 4: a tap is unrolled, with its weights straight from memory and one tap
// ahead in registers, tile by tile, the folds between the tiles.  A tap so short has a fold, new addresses and masks for every 4 to 16
// matrix instructions, and this order hides them best; with more steps the ring wins (below).  us a call, steps in a loop with a ring
// -> this:
//     per-pixel scales  16 x 24 x 53 x 192 13.5 -> 12.7, 3 x 64 x 64 x 384 -> 96 (a slice at a time) 18.5 -> 16.5
//     one scale         5 x 54 x 54 x 64 10.1 -> 7.9, 24 x 33 x 22 x 192 15.5 -> 12.4, 9 x 32 x 46 x 576 -> 264 (a slice at a time) 35.9 -> 28.0
//     width axis        4 x 49 x 48 x 192, block 16 14.7 -> 12.4;   8 bits  12 x 23 x 17 x 384 -> 392 (a slice at a time) 20.2 -> 18.2
// TAIL: channel counts that are no multiple of 64 too.  A form of its own, because the branches cost layers of whole steps 1 to 2 %, up to
// 4 (2 x 24 x 40 x 640 14.8 -> 15.4 us, one scale 1 x 6 x 200 x 960 -> 40 23.8 -> 24.6), and a loop of its own in the same kernel costs the sums of
// codes 2.
template <int OUT, int KIND, int RING, int NS, bool TAIL>
__global__ __launch_bounds__(512, 2) void resident_kernel(ResidentArgs) {
    constexpr bool WHOLE_TAPS = KIND == kResWholeTaps;   // (see the offset of the weights above)
    constexpr bool BYTES = KIND == kResBytes, FOLD = KIND == kResPerTap || WHOLE_TAPS || BYTES, INT_TAPS = OUT == kOutI32 && FOLD;
    constexpr int TAPS = 9, NT = 4;
    // planes in memory, operand planes in LDS (BYTES: the two 32-channel halves of a step) and of the weights
    constexpr int IN = KIND == kResPlanes ? 3 : BYTES ? 2 : 1, PL = KIND == kResPlanes || BYTES ? 2 : 1, WP = BYTES ? 2 : 1;
    constexpr int STEP = BYTES ? 64 : 32;   // bytes of a step of 64 codes
    // Steps of an item of the fill, and items whose loads are in flight.  Items of one step have an address, a branch and an atomic sum
    // for every 16 bytes a lane; us a call, items of one step, four in flight -> of three: one scale 2 x 23 x 23 x 576 13.9 -> 12.8,
    // per-pixel scales 7 x 12 x 8 x 768 -> 216 17.9 -> 17.0.  The forms of three planes (2 .. 10 % slower with three steps) and of 8 bits
    // (eight waves, 2 %) keep to one.
    constexpr int PIECES = NS ? NS : IN == 1 ? 3 : 1, AHEAD = 2;
    using Out = typename OutT<OUT>::type;
    using Operand = std::conditional_t<BYTES, v4i, v8i>;
    using Acc = std::conditional_t<BYTES, v16i, v16f>;
    constexpr float UNIT = BYTES ? 1.0f : 64.0f;   // a product of two codes is 1 / UNIT in the accumulators
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ResidentArgs a;
    start_args(a);
    auto row_bytes = [](const auto &a) { return BYTES ? a.k : a.k >> 1; };   // of a pixel's codes, and of a channel's for one tap

    // workgroup b runs on XCD b % 8: every XCD gets a contiguous run of tiles
    const uint32_t nwg = a.tiles, xcd = blockIdx.x & 7, q8 = nwg >> 3, r8 = nwg & 7;
    const uint32_t tile = xcd * q8 + (xcd < r8 ? xcd : r8) + (blockIdx.x >> 3);
    const uint32_t slow_i = hq::div_magic31(tile, a.fast, a.d_magic, a.d_shift), fast_i = tile - slow_i * a.fast;
    const uint32_t px_tile = a.ch_major ? fast_i : slow_i, p0 = px_tile << (7 + a.xw_log2);
    const int c_wg = static_cast<int>(a.ch_major ? slow_i : fast_i) * a.cb * 32;
    const int blocks = min(a.cb, (a.n - c_wg + 31) / 32);   // channel blocks of this workgroup

    struct Tables {
        float *sx;         // [tap][pixel] scales
        float *corr;       // [pixel]
        int *mask;         // [pixel]
        float *rowscale;   // [row]
        int *sum;          // [row] code sums of the resident steps
        float *sw, *bias;  // [channel]
        short *part;       // WHOLE_TAPS: code sums [three resident steps][row]
    };
    auto tables_of = [&](const auto &a) {
        const int px = 128 << a.xw_log2;
        Tables t;
        t.sx = reinterpret_cast<float *>(lds + a.tables);
        t.corr = t.sx + (FOLD ? TAPS : 0) * px;
        t.mask = reinterpret_cast<int *>(t.corr + px);
        t.rowscale = reinterpret_cast<float *>(t.mask + px);
        t.sum = reinterpret_cast<int *>(t.rowscale + a.rows);
        t.sw = reinterpret_cast<float *>(t.sum + a.rows);
        t.bias = t.sw + a.cb * 32;
        t.part = reinterpret_cast<short *>(t.bias + a.cb * 32);
        return t;
    };

    // ---- phases: tasks and shares ---------------------------------------------------------------------------
    // tasks first .. first + (nw >> kl) - 1, each by 1 << kl waves; wave wv has task first + wv >> kl, share wv mod
    int left = blocks << a.xw_log2, first = 0, kl = 0;
    const int nw = a.waves;
    auto shrink = [&]() {   // (4 or 8 waves)
        kl = left * 8 < nw * 2 ? 3 : left * 4 < nw * 2 ? 2 : left < nw ? 1 : 0;
    };
    shrink();
    int c0 = 0, px_l = 0;    // first channel, first pixel (local)
    int s0 = 0, ns = a.chunk;   // resident steps s0 .. s0 + ns - 1
    int tap0 = 0, step0 = 0, share_steps = 0;   // this wave's share: first tap and resident step, steps

    // ---- weights: from memory into the wave's ring in LDS, R steps ahead --------------------------------------
    // A step's 32 rows of 32 bytes (BYTES: 64) are fetched by neighbouring lanes piece by piece, which takes the address
    // path 22 clocks a KiB; loads straight into the operand's lanes (16 rows in every 16 lanes) take 37, more than the matrix
    // instructions that the KiB feeds.  In rows 8..15 mod 16 (BYTES: 4..7, 8..11, 12..15) the pieces change places, so that
    // the operand reads meet no bank conflict.  Every step requests one (past the share's end what follows there), so the
    // number of requests in flight is always the same.
    constexpr int R = RING, SLOT = resident_slot_bytes(KIND), DMAS = SLOT / 1024;
    const uint32_t w_bytes = static_cast<uint32_t>(a.n) * (TAPS * row_bytes(a));
    const v4i w_buf = buffer_words(a.wq, w_bytes);
    constexpr int UNROLL = RING ? RING : 3;   // steps of a group (below): a ring's slots come round
    uint32_t w_row[DMAS];    // this lane's pieces: offset of the position requested last (without a ring: [0], its operand's row)
    // where this lane's operand pieces lie in the slots, and the slots themselves; [0]: filled next
    int r_piece[RING ? RING : 1][WP];
    uint32_t r_slot[RING ? RING : 1];
    uint32_t w_gap = 0;      // from the last of a tap's resident steps to the first of the next, less a step
    int w_left = 0;          // steps to request before that
    v4i raw[WP];             // weights of the next step (BYTES: of this step) as they lie in memory
    auto skip_gap = [&]() {
#pragma unroll
        for (int j = 0; j < DMAS; ++j) w_row[j] += w_gap;
        w_left = ns;
    };
    auto request = [&](int slot) {   // the next position into a slot
        if constexpr (RING > 0) {
#pragma unroll
            for (int j = 0; j < DMAS; ++j) load_to_ring<STEP>(w_buf, w_row[j], r_slot[slot] + j * 1024);
        }
    };
    auto take = [&](int slot) {      // raw <- the weights in a slot; R - 1 steps were requested after them
        if constexpr (RING > 0) {
            wait_vmem<(R - 1) * DMAS>();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < WP; ++i) raw[i] = lds_v4i(r_piece[slot][i]);
        } else {
            const __amdgpu_buffer_rsrc_t buf = buffer_of(a.wq, w_bytes);
            if (w_left == 0) skip_gap();
            --w_left;
            w_row[0] += STEP;
#pragma unroll
            for (int i = 0; i < WP; ++i) raw[i] = buffer_load16(buf, w_row[0], i * 32);
        }
    };
    auto request_next = [&](int slot) {   // wherever in a tap it is
        if constexpr (RING > 0) {
            if (w_left == 0) skip_gap();
            --w_left;
            request(slot);
        }
    };
    v4i raw_tap[WP][NS ? NS : 1];   // NS: weights of the next tap
    auto take_tap = [&](int tap, int tap_bytes) {
        const __amdgpu_buffer_rsrc_t buf = buffer_of(a.wq, w_bytes);
#pragma unroll
        for (int k = 0; k < NS; ++k)
#pragma unroll
            for (int i = 0; i < WP; ++i)
                raw_tap[i][k] = buffer_load16(buf, w_row[0], static_cast<uint32_t>(tap * tap_bytes + (s0 + k) * STEP + i * 32));
    };
    auto begin_task = [&](const auto &a) {
        const int lane = thread_again() & 63, l = lane & 31, h = lane >> 5, cb = row_bytes(a);
        const int task = first + (wv >> kl), share = wv & ((1 << kl) - 1);
        px_l = (task & ((1 << a.xw_log2) - 1)) * 128;
        c0 = c_wg + (task >> a.xw_log2) * 32;
        auto row_of = [&](int i) {
            const int co = c0 + tile_row_to_channel(i);
            return static_cast<uint32_t>(co < a.n ? co : a.n - 1) * (TAPS * cb);
        };
#pragma unroll
        for (int j = 0; j < DMAS; ++j) {
            const int row = BYTES ? j * 16 + (lane >> 2) : lane >> 1;
            w_row[j] = row_of(row) + (BYTES ? (lane & 3) ^ ((row >> 2) & 3) : (lane & 1) ^ ((row >> 3) & 1)) * 16;
        }
        if constexpr (RING == 0) w_row[0] = row_of(l) + h * 16;
        // (A tap that two waves share is folded twice: fp32 results are cut at every third step of a tap only, where WHOLE_TAPS has code sums.  So are chunks and
        // taps whose last step is not whole, for the sake of the groups of steps.)
        struct Cut { int tap, step; };
        auto cut = [&](int of) {
            if constexpr (NS > 0) {
                return Cut{of * TAPS >> kl, 0};
            } else if (OUT == kOutF32 || cb != ns * STEP) {
                const int grains = (ns + 2) / 3, at = of * (TAPS * grains) >> kl, tap = quotient(at, (ns == a.chunk ? a.inverses : a.inverses_last) >> 16);
                return Cut{tap, (at - tap * grains) * 3};
            } else {
                const int at = of * (TAPS * ns) >> kl, tap = quotient(at, (ns == a.chunk ? a.inverses : a.inverses_last) & 0xFFFF);
                return Cut{tap, at - tap * ns};
            }
        };
        const Cut from = cut(share), to = cut(share + 1);
        tap0 = from.tap;
        step0 = from.step;
        share_steps = (to.tap - from.tap) * ns + to.step - from.step;
        if constexpr (NS > 0) {
            take_tap(tap0, cb);
        } else {
#pragma unroll
            for (int j = 0; j < DMAS; ++j) w_row[j] += tap0 * cb + (s0 + step0 - 1) * STEP;
            w_gap = cb - ns * STEP;
            w_left = ns - step0;
        }
        if constexpr (RING > 0) {
            const uint32_t ring = lds_address(lds) + a.ring + wv * a.ring_stride;   // (uniform)
#pragma unroll
            for (int i = 0; i < R; ++i) {
                r_slot[i] = ring + i * SLOT;
#pragma unroll
                for (int j = 0; j < WP; ++j)
                    r_piece[i][j] = static_cast<int>(r_slot[i]) +
                                    (BYTES ? l * 64 + ((2 * j + h) ^ ((l >> 2) & 3)) * 16 : l * 32 + (h ^ ((l >> 3) & 1)) * 16);
                request_next(i);
            }
        }
    };

    // ---- activation tile: packed codes -> signed 6-bit fields ------------------------------------------------
    // Wave items (32 rows, PIECES steps): lane = (row, lane half), a 16-byte piece of each step; the code sum of a row's item is that of
    // two neighbouring lanes.  Neighbouring waves take the steps of the same rows.
    struct Item { int step, row; };
    // set by begin_fill
    int nw_step = 0, nw_row = 0, row_steps = 0;   // nw items on; steps of a row, up to a whole item
    int f_row = 0, f_half = 0, row_span = 0, rows = 0;
    uint32_t f_off = 0, f_row_bytes = 0, plane_bytes = 0;
    const uint8_t *x_codes = nullptr;
    uint32_t part8 = 0;
    int tail = 0, tail_step = 0;   // TAIL: packed dwords of the last step if it is not whole, and which it is
    int in_planes = 0;
    int *f_sum = nullptr;     // code sums
    short *f_part = nullptr;
    auto next = [&](Item &i) {
        i.step += nw_step;
        i.row += nw_row;
        if (NS == 0 && i.step >= row_steps) {
            i.step -= row_steps;
            i.row += 32;
        }
    };
    auto fill_load = [&](v4i (&p)[IN][PIECES], const Item &item) {
        if (item.row >= row_span) return;
        // (rows outside the tensor wrap or lie beyond the bound and read as zeros; they are never used)
        const uint32_t off = f_off + item.row * f_row_bytes;
        const __amdgpu_buffer_rsrc_t x_buf = buffer_of(x_codes, BYTES ? plane_bytes : IN * plane_bytes);
#pragma unroll
        for (int i = 0; i < IN; ++i)
#pragma unroll
            for (int k = 0; k < PIECES; ++k) {
                if (PIECES > 1 && NS == 0 && item.step + k >= ns) continue;
                if (IN < 3 || i < in_planes) p[i][k] = buffer_load16(x_buf, off, i * (BYTES ? 32u : plane_bytes) + (s0 + item.step + k) * STEP);
                else p[i][k] = v4i{0, 0, 0, 0};
            }
    };
    auto cut_tail = [&](v4i (&p)[IN][PIECES], const Item &item) {   // the rest are codes of zero
        if constexpr (TAIL) {   // (if the last step is whole, the one after it, which is in no item)
#pragma unroll
            for (int k = 0; k < PIECES; ++k)
                if (item.step + k == tail_step) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) p[0][k][e] = f_half * 4 + e < tail ? p[0][k][e] : 0;
                }
        }
    };
    auto fill_store = [&](const v4i (&p)[IN][PIECES], const Item &item) {
        const int row = item.row + f_row;
        int sum = 0;
        if (row < rows - 1) {
#pragma unroll
            for (int k = 0; k < PIECES; ++k) {
                if (PIECES > 1 && NS == 0 && item.step + k >= ns) break;
                auto at = [&](int plane) { return (((item.step + k) * PL + plane) * 2 + f_half) * rows + row; };
                if constexpr (BYTES) {
#pragma unroll
                    for (int i = 0; i < PL; ++i) *reinterpret_cast<v4i *>(lds + at(i) * 16) = p[i][k];
                } else {
                    auto codes = [&](const v4i &v, int s) {
                        return sum_codes8(v.x, sum_codes8(v.y, sum_codes8(v.z, sum_codes8(v.w, s))));
                    };
                    auto put = [&](int plane, const int (&d)[6]) {
                        *reinterpret_cast<v4i *>(lds + at(plane) * 16) = v4i{d[0], d[1], d[2], d[3]};
                        *reinterpret_cast<int2 *>(lds + part8 + at(plane) * 8) = int2{d[4], d[5]};
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
        }
        if constexpr (!BYTES) {
            sum += __builtin_amdgcn_mov_dpp(sum, 0xB1, 0xF, 0xF, true);   // the other half of the row (lanes 1,0,3,2)
            if (f_half == 0 && row < rows - 1) {
                if constexpr (WHOLE_TAPS) f_part[item.step / PIECES * rows + row] = static_cast<short>(sum);
                else atomicAdd(&f_sum[row], sum);
            }
        }
    };

    // All first loads are requested before any is waited for (a first use costs a trip to HBM).
    v4i p[AHEAD][IN][PIECES];
    Item load_item{}, store_item{};
    auto begin_fill = [&](const auto &a) {
        const int lane = thread_again() & 63;
        const uint32_t cb = row_bytes(a);
        f_row = lane >> 1;
        f_half = lane & 1;
        rows = a.rows;
        row_span = ((128 << a.xw_log2) + 2 * (a.w + 1) + 31) & ~31;
        x_codes = a.xq;
        f_row_bytes = cb;
        plane_bytes = a.pixels * cb;
        in_planes = a.in_planes;
        part8 = a.part8;
        tail = (a.k & 63) >> 3;
        tail_step = (a.k >> 6) - s0;
        const Tables table = tables_of(a);
        f_sum = table.sum;
        f_part = table.part;
        f_off = (p0 - (a.w + 1) + f_row) * cb + f_half * 16;
        const int of_rows = NS ? 1 : (ns + PIECES - 1) / PIECES;   // items of 32 rows
        const uint32_t inverses = ns == a.chunk ? a.inverses : a.inverses_last, inv = PIECES == 1 ? inverses & 0xFFFF : inverses >> 16;
        const int nw_q = NS ? nw : quotient(nw, inv), wv_q = NS ? wv : quotient(wv, inv);
        row_steps = of_rows * PIECES;
        nw_row = nw_q * 32;
        nw_step = (nw - nw_q * of_rows) * PIECES;
        load_item = store_item = Item{(wv - wv_q * of_rows) * PIECES, wv_q * 32};
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
#pragma unroll
            for (int j = 0; j < IN * PIECES; ++j) asm("" : "=v"(p[i][j / PIECES][j % PIECES]));   // (no register holds the old ones meanwhile)
            fill_load(p[i], load_item);
            next(load_item);
        }
    };
    begin_fill(a);
    begin_task(a);
    constexpr bool ROW_SCALES = FOLD && !INT_TAPS, SUMS = !BYTES && !WHOLE_TAPS;
    auto row_scale = [&](const auto &a, int i) {
        const int64_t last = a.pixels - 1u;
        int64_t pix = static_cast<int64_t>(p0) - (a.w + 1) + i;
        pix = pix < 0 ? 0 : (pix > last ? last : pix);
        return a.sx[pix];
    };
    float t_scale[2] = {}, t_sw = 0.f;
    Out t_bias{};
    {
        const int tid = thread_again(), nt = nw * 64;
        if constexpr (ROW_SCALES) {
            t_scale[0] = row_scale(a, tid);
            t_scale[1] = row_scale(a, tid + nt);
        }
        if constexpr (OUT != kOutI32) {
            const int c = c_wg + tid < a.n ? c_wg + tid : a.n - 1;
            t_sw = a.sw[c];
            t_bias = static_cast<const Out *>(a.bias ? a.bias : a.sw)[c];   // (without a bias: not used; a branch would wait for it)
        }
    }
    auto clear_sums = [&]() {
        if constexpr (SUMS) {
            for (int i = thread_again(); i < rows; i += nw * 64) f_sum[i] = 0;
            lds_barrier();   // the code sums are zero before they are added to
        }
    };
    clear_sums();

    int touched = 0;     // (see below)
    v16f sum[NT];        // the accumulators themselves, or (FOLD) fp32 combinations of per-tap sums
    for (;;) {           // chunks of resident steps
        while (store_item.row < row_span) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (store_item.row >= row_span) break;
                cut_tail(p[i], store_item);
                fill_store(p[i], store_item);
                next(store_item);
                fill_load(p[i], load_item);
                next(load_item);
            }
        }
        KernelArgs &a = args_again();
        const int tid = thread_again(), nt = nw * 64, px_wg = 128 << a.xw_log2, halo = a.w + 1;
        const uint32_t cb = row_bytes(a);
        const Tables table = tables_of(a);
        if (s0 == 0) {
            // The weights of the workgroup's channels start their way into the L2: from HBM they would take longer than the loop over
            // steps looks ahead.  A word of every line; workgroups that share the channels take an eighth each.  us a call, weights not in
            // L2, without -> with, no ring: 1 x 63 x 63 x 768 28.3 -> 25.9.  (Forms of two operand
            // planes, without a ring: 8 bits 1.5 % slower with it, 16 x 16 x 16 x 576 on the width axis 29.3 -> 29.7.)
            const uint32_t line = ((px_tile & 7) * nt + tid) * 128u, size = static_cast<uint32_t>(min(blocks * 32, a.n - c_wg)) * (TAPS * cb);
            if (NS == 0 && (RING > 0 || PL == 1) && line < size) touched = *reinterpret_cast<const int *>(a.wq + static_cast<uint32_t>(c_wg) * (TAPS * cb) + line);
            if constexpr (ROW_SCALES) {
                if (tid < rows) table.rowscale[tid] = t_scale[0];
                if (tid + nt < rows) table.rowscale[tid + nt] = t_scale[1];
                for (int i = tid + 2 * nt; i < rows; i += nt) table.rowscale[i] = row_scale(a, i);
            }
            if constexpr (OUT != kOutI32) {
                if (tid < blocks * 32) {
                    table.sw[tid] = t_sw;
                    table.bias[tid] = a.bias ? to_float(t_bias) : 0.f;
                }
                for (int i = tid + nt; i < blocks * 32; i += nt) {
                    const int c = c_wg + i < a.n ? c_wg + i : a.n - 1;
                    table.sw[i] = a.sw[c];
                    table.bias[i] = a.bias ? to_float(static_cast<const Out *>(a.bias)[c]) : 0.f;
                }
            }
        }
        lds_barrier();
        // tables of the pixels: tap masks, scales under the taps, corrections
        if constexpr (NS == 0 || KIND == kResPerTap || WHOLE_TAPS) {   // a lane has one row of the window, four lanes a pixel
            for (int j = tid; j < 4 * px_wg; j += nt) {
                const int r = j & 3, i = j >> 2;   // (r == 3: nothing)
                const uint32_t pix = p0 + i;
                const uint32_t line = hq::div_magic31(pix, a.w, a.w_magic, a.w_shift);
                const int ow = static_cast<int>(pix - line * a.w);
                const int oh = static_cast<int>(line - hq::div_magic31(line, a.h, a.h_magic, a.h_shift) * a.h);
                const int cm = (ow > 0 ? 1 : 0) | 2 | (ow + 1 < a.w ? 4 : 0);
                int mask = (oh > 0 ? cm : 0) | (cm << 3) | (oh + 1 < a.h ? cm << 6 : 0);
                if (pix >= a.pixels) mask = 0;
                if (r == 0) table.mask[i] = mask;
                float corr = 0.f;
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    if (r == 3) break;
                    const int t = 3 * r + s, row = halo + i + (r - 1) * a.w + (s - 1);
                    const bool in = (mask >> t) & 1;
                    if constexpr (ROW_SCALES) {
                        const float scale = in ? table.rowscale[row] : 0.f;
                        table.sx[t * px_wg + i] = scale;
                        if constexpr (SUMS) corr = fmaf(scale * (8.0f / UNIT), static_cast<float>(table.sum[row]), corr);
                    } else if (SUMS && in) {
                        corr += (8.0f / UNIT) * static_cast<float>(table.sum[row]);
                    }
                }
                corr += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, corr), 0xB1, 0xF, 0xF, true));   // lanes 1,0,3,2
                corr += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, corr), 0x4E, 0xF, 0xF, true));   // lanes 2,3,0,1
                if (r == 0) table.corr[i] = corr;
            }
        } else {   // a lane has a pixel: as fast for 128 pixels, faster for 256 (with per-pixel scales of 4-bit codes its registers spill)
            for (int i = tid; i < px_wg; i += nt) {
                const uint32_t pix = p0 + i;
                const uint32_t line = hq::div_magic31(pix, a.w, a.w_magic, a.w_shift);
                const int ow = static_cast<int>(pix - line * a.w);
                const int oh = static_cast<int>(line - hq::div_magic31(line, a.h, a.h_magic, a.h_shift) * a.h);
                const int cm = (ow > 0 ? 1 : 0) | 2 | (ow + 1 < a.w ? 4 : 0);
                int mask = (oh > 0 ? cm : 0) | (cm << 3) | (oh + 1 < a.h ? cm << 6 : 0);
                if (pix >= a.pixels) mask = 0;
                table.mask[i] = mask;
                float corr = 0.f;
#pragma unroll
                for (int t = 0; t < TAPS; ++t) {
                    const int row = halo + i + (t / 3 - 1) * a.w + (t % 3 - 1);
                    const bool in = (mask >> t) & 1;
                    if constexpr (ROW_SCALES) table.sx[t * px_wg + i] = in ? table.rowscale[row] : 0.f;
                    else if (SUMS && in) corr += (8.0f / UNIT) * static_cast<float>(table.sum[row]);
                }
                if constexpr (SUMS) table.corr[i] = corr;
            }
        }
        if constexpr (WHOLE_TAPS && NS == 0) {   // code sums of three steps -> of all resident steps up to them
            for (int i = tid; i < px_wg + 2 * halo; i += nt) {
                int of = table.part[i];
                for (int k = PIECES; k < ns; k += PIECES) {
                    of += table.part[k / PIECES * rows + i];
                    table.part[k / PIECES * rows + i] = static_cast<short>(of);
                }
            }
        }
        lds_barrier();

        for (;;) {   // phases
            KernelArgs &a = args_again();
            const int lane = thread_again() & 63, l = lane & 31, h = lane >> 5, rows = a.rows;
            const Tables table = tables_of(a);
            const float *const s_sx = table.sx;
            const int px_wg = 128 << a.xw_log2;
            int mask[NT];   // kResSum / INT_TAPS: taps inside the image, for the pixels of the four tiles
            if constexpr (!FOLD || INT_TAPS) {
#pragma unroll
                for (int t = 0; t < NT; ++t) mask[t] = table.mask[px_l + t * 32 + l];
            }
            // the sums start from minus the correction for the weights' offset
            const bool corrects = SUMS && !INT_TAPS && (wv & ((1 << kl) - 1)) == 0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                float from = 0.f;
                if (corrects) {
                    const int i = px_l + t * 32 + l;
                    from = -table.corr[i];
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) sum[t][i] = s0 == 0 ? from : sum[t][i] + from;
            }
            const int lane_row = px_l + l + a.w + 1;

            if constexpr (NS > 0) {
                // While the MFMAs of a tile run, the next one is on its way from LDS and the sums of the one before are folded; the next
                // tap's weights are requested as soon as this one's are expanded.
                const Fp6Masks masks;
                const int step16 = rows * (PL * 32), step8 = rows * (PL * 16), plane16 = rows * 32, plane8 = rows * 16;
                int tap = tap0;
                const int tap_end = tap0 + share_steps / NS, tap_bytes = row_bytes(a);
                struct Base { int b16, b8; };
                auto row_shift = [&](int tap) { return (tap / 3 - 1) * a.w + tap % 3 - 1; };
                auto base_of = [&](int tap) {
                    const int at = lane_row + row_shift(tap) + h * rows;
                    return Base{static_cast<int>(lds_address(lds)) + at * 16, static_cast<int>(lds_address(lds) + a.part8) + at * 8};
                };
                auto load_tile = [&](Operand (&b)[NS], const Base &base, int t, int plane) {
#pragma unroll
                    for (int k = 0; k < NS; ++k) {
                        const v4i lo = lds_v4i(base.b16 + k * step16 + plane * plane16, t * 512);
                        if constexpr (BYTES) {
                            b[k] = lo;
                        } else {
                            const v2i hi = lds_v2i(base.b8 + k * step8 + plane * plane8, t * 256);
                            b[k] = v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, 0, 0};
                        }
                    }
                };
                const v4h minus = h ? v4h{} : v4h{-0.125f16, -128.0f16, 0, 0};
                Base base = base_of(tap);
                Operand wop[WP][NS], b[2][NS];
                load_tile(b[0], base, 0, 0);
                for (; tap < tap_end; ++tap) {
                    const int tap1 = tap + 1 < tap_end ? tap + 1 : tap;   // (the last one's operands are requested twice)
                    const Base base1 = base_of(tap1);
#pragma unroll
                    for (int k = 0; k < NS; ++k) {
                        if constexpr (BYTES) {
#pragma unroll
                            for (int i = 0; i < WP; ++i) wop[i][k] = raw_tap[i][k];
                        } else {
                            int d[6];
                            fp6_offset16(masks, raw_tap[0][k].x, raw_tap[0][k].y, d[0], d[1], d[2]);
                            fp6_offset16(masks, raw_tap[0][k].z, raw_tap[0][k].w, d[3], d[4], d[5]);
                            wop[0][k] = v8i{d[0], d[1], d[2], d[3], d[4], d[5], 0, 0};
                        }
                    }
                    take_tap(tap1, tap_bytes);
                    float scale[NT];
                    int codes[NT], inside[NT];   // (as below)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if constexpr (ROW_SCALES) scale[t] = s_sx[tap * px_wg + px_l + t * 32 + l];
                        if constexpr (WHOLE_TAPS) codes[t] = table.part[lane_row + row_shift(tap) + t * 32];
                        if constexpr (!FOLD) inside[t] = (mask[t] >> tap) & 1 ? 127 : 0;
                    }
                    Acc acc[2];
                    auto fold = [&](int t) {
                        if constexpr (FOLD) {
#pragma unroll
                            for (int i = 0; i < 16; ++i) sum[t][i] = fmaf(scale[t], static_cast<float>(acc[t & 1][i]), sum[t][i]);
                        }
                    };
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if constexpr (WHOLE_TAPS) acc[t & 1] = __builtin_bit_cast(Acc, minus_eighth_of(minus, codes[t]));
                        else if constexpr (FOLD) acc[t & 1] = Acc{};
#pragma unroll
                        for (int plane = 0; plane < PL; ++plane) {
                            const int now = t * PL + plane, next = now + 1;
                            if (next < NT * PL) load_tile(b[next & 1], base, next / PL, next % PL);
                            else load_tile(b[0], base1, 0, 0);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int k = 0; k < NS; ++k) {
                                if constexpr (BYTES) acc[t & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wop[plane][k], b[now & 1][k], acc[t & 1], 0, 0, 0);
                                else if constexpr (FOLD) acc[t & 1] = mfma_fp6(wop[0][k], b[now & 1][k], acc[t & 1]);
                                else sum[t] = mfma_fp6_scaled(wop[0][k], b[now & 1][k], sum[t], plane ? 131 : 127, inside[t]);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                            if (t > 0 && plane == 0) fold(t - 1);
                        }
                    }
                    fold(NT - 1);
                    base = base1;
                }
            } else {
                int tap = tap0, k = step0;
                // LDS addresses of the operands of the step at work: the 16- and the 8-byte parts of this lane's row of tile 0; the
                // other tiles lie at fixed distances.
                const int step16 = rows * (PL * 32), plane16 = rows * 32, plane8 = rows * 16;
                auto row_shift = [&](int tap) { return (tap / 3 - 1) * a.w + tap % 3 - 1; };
                const int first_row = lane_row + row_shift(tap) + h * rows;
                int b16 = static_cast<int>(lds_address(lds)) + first_row * 16 + k * step16;
                int b8 = static_cast<int>(lds_address(lds) + a.part8) + first_row * 8 + (k * step16 >> 1);
                Operand b[NT][PL];
                int wop[UNROLL][6];   // weights of this step and, at the next place, of the next one
                auto load_tile = [&](int t) {
#pragma unroll
                    for (int plane = 0; plane < PL; ++plane) {
                        const v4i lo = lds_v4i(b16 + plane * plane16, t * 512);
                        if constexpr (BYTES) {
                            b[t][plane] = lo;
                        } else {
                            const v2i hi = lds_v2i(b8 + plane * plane8, t * 256);
                            b[t][plane] = v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, 0, 0};
                        }
                    }
                };
                const Fp6Masks masks;
                auto expand_weights = [&](const v4i &r, int pair, int (&o)[6]) {
                    if constexpr (!BYTES) {
                        int *const d = o + 3 * pair;
                        if (pair == 0) fp6_offset16(masks, r.x, r.y, d[0], d[1], d[2]);
                        else fp6_offset16(masks, r.z, r.w, d[0], d[1], d[2]);
                        asm volatile("" : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]));   // (here, between two matrix instructions)
                    }
                };

                Acc acc[NT];              // FOLD: the sums of the tap at work
                const v4h minus = h ? v4h{} : v4h{-0.125f16, -128.0f16, 0, 0};
                auto codes_upto = [&](int step, int t) {   // WHOLE_TAPS
                    return static_cast<int>(table.part[step / PIECES * rows + lane_row + (tap / 3 - 1) * a.w + tap % 3 - 1 + t * 32]);
                };
                // A step.  Right after the matrix instructions of a tile the tile's operands of the next step are requested, into the
                // registers that have just been read; the next step's weights are expanded in between, and their slot of the
                // ring is filled again.  on: from this step's operands to the next one's.
                int inside[NT];   // !FOLD: block exponents: 2^0, or for taps outside the image one that leaves nothing
                auto step = [&](auto STARTS, auto PLACE, int on, auto fill) {   // the tap's sums start here
                    constexpr bool starts = decltype(STARTS)::value;
                    constexpr int place = decltype(PLACE)::value, next = (place + 1) % UNROLL;
                    b16 += on;
                    b8 += on >> 1;
                    v4i now[WP];
#pragma unroll
                    for (int i = 0; i < WP; ++i) now[i] = raw[i];
                    const int (&o)[6] = wop[place];
                    const v8i weights = v8i{o[0], o[1], o[2], o[3], o[4], o[5], 0, 0};
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if constexpr (BYTES) {
                            Acc c = starts ? Acc{} : acc[t];
#pragma unroll
                            for (int i = 0; i < PL; ++i) c = __builtin_amdgcn_mfma_i32_32x32x32_i8(now[i], b[t][i], c, 0, 0, 0);
                            acc[t] = c;
                        } else if constexpr (FOLD) {
                            acc[t] = mfma_fp6(weights, b[t][0], starts && !WHOLE_TAPS ? Acc{} : acc[t]);
                        } else {
                            sum[t] = mfma_fp6_scaled(weights, b[t][0], sum[t], 127, inside[t]);
                            if constexpr (PL == 2) sum[t] = mfma_fp6_scaled(weights, b[t][PL - 1], sum[t], 131, inside[t]);   // (x 2^4)
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        load_tile(t);
                        if (t == 0) expand_weights(now[0], 0, wop[next]);
                        if (t == 1) expand_weights(now[0], 1, wop[next]);
                        if (t == (BYTES ? 0 : 2)) {
                            fill(place);   // (the slot of the weights that have just been used, or expanded)
                            take(next);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
                auto rotate = [&]() {   // the slots go on by one
                    if constexpr (RING > 0) {
                        const uint32_t slot = r_slot[0];
#pragma unroll
                        for (int i = 0; i + 1 < R; ++i) r_slot[i] = r_slot[i + 1];
                        r_slot[R - 1] = slot;
#pragma unroll
                        for (int j = 0; j < WP; ++j) {
                            const int piece = r_piece[0][j];
#pragma unroll
                            for (int i = 0; i + 1 < R; ++i) r_piece[i][j] = r_piece[i + 1][j];
                            r_piece[R - 1][j] = piece;
                        }
                    }
                };
                // A step by itself: the next one's weights come to the first place again.
                auto single = [&](int on) {
                    step(std::false_type{}, std::integral_constant<int, 0>{}, on, request_next);
#pragma unroll
                    for (int i = 0; i < 6; ++i) wop[0][i] = wop[1][i];
                    rotate();
                };
                // UNROLL steps, as many as are left in the tap or a multiple of them: the requests, ahead by UNROLL + 1 steps (BYTES:
                // UNROLL), come to the end of a tap with the last (first) step of a group or not at all.
                auto group = [&](auto STARTS, int on) {
                    constexpr int CROSSES = BYTES ? 0 : UNROLL - 1;
                    auto fill = [&](int place) {
                        if (RING > 0 && place == CROSSES) {
                            const bool crosses = w_left == CROSSES;
#pragma unroll
                            for (int j = 0; j < DMAS; ++j) w_row[j] += crosses ? w_gap : 0;
                            w_left += (crosses ? ns : 0) - UNROLL;
                        }
                        request(place);
                    };
                    step(STARTS, std::integral_constant<int, 0>{}, step16, fill);
                    if constexpr (UNROLL == 3) step(std::false_type{}, std::integral_constant<int, 1>{}, step16, fill);
                    step(std::false_type{}, std::integral_constant<int, UNROLL - 1>{}, on, fill);
                };
#pragma unroll
                for (int t = 0; t < NT; ++t) load_tile(t);
                take(0);
                if constexpr (!BYTES) {
                    expand_weights(raw[0], 0, wop[0]);
                    expand_weights(raw[0], 1, wop[0]);
                    request_next(0);
                    take(1);
                    rotate();
                }
                // (in the order of memory the requests cross from tap to tap unnoticed)
                const bool groups = RING == 0 || w_gap == 0 || (UNROLL == 3 && ns % 3 == 0);
                for (int to_go = share_steps; to_go > 0;) {   // taps
                    const int n = min(ns - k, to_go);
                    // from the last step to the next tap's first (past the last tap: the same operands again, not used)
                    const int over = tap + 1 < TAPS ? (row_shift(tap + 1) - row_shift(tap)) * 16 - (k + n - 1) * step16 : 0;
                    float scale[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if constexpr (ROW_SCALES) scale[t] = s_sx[tap * px_wg + px_l + t * 32 + l];
                        if constexpr (WHOLE_TAPS)   // the sums of a tap start with the offset of the steps that this wave will add
                            acc[t] = __builtin_bit_cast(Acc, minus_eighth_of(minus, codes_upto(k + n - 1, t) - (k ? codes_upto(k - 1, t) : 0)));
                    }
                    if constexpr (!FOLD) {
#pragma unroll
                        for (int t = 0; t < NT; ++t) inside[t] = (mask[t] >> tap) & 1 ? 127 : 0;
                    }
                    int left = n;
                    if constexpr (FOLD && !WHOLE_TAPS) {
                        if (n >= UNROLL && groups) {
                            group(std::true_type{}, left == UNROLL ? over : step16);
                            left -= UNROLL;
                        } else {
#pragma unroll
                            for (int t = 0; t < NT; ++t) acc[t] = Acc{};
                        }
                    }
                    if (groups) {
#pragma unroll 1
                        for (; left >= UNROLL; left -= UNROLL) group(std::false_type{}, left == UNROLL ? over : step16);
                    }
#pragma unroll 1
                    for (; left > 0; --left) single(left == 1 ? over : step16);
                    if constexpr (INT_TAPS) {
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            const uint32_t pix = p0 + px_l + t * 32 + l;
                            if (!((mask[t] >> tap) & 1)) continue;
                            const int row = lane_row + (tap / 3 - 1) * a.w + tap % 3 - 1 + t * 32;
                            const int extra = !BYTES && k == 0 ? 8 * table.sum[row] : 0;
                            int *dst = static_cast<int *>(a.y) + (static_cast<uint64_t>(pix) * 9 + tap) * a.n;
#pragma unroll
                            for (int i = 0; i < 16; ++i) {
                                const int c = c0 + 16 * h + i;
                                if (c < a.n) atomicAdd(dst + c, static_cast<int>(acc[t][i] * static_cast<decltype(acc[t][i] + 0)>(UNIT)) - extra);
                            }
                        }
                    } else if constexpr (FOLD) {
#pragma unroll
                        for (int t = 0; t < NT; ++t)
#pragma unroll
                            for (int i = 0; i < 16; ++i) sum[t][i] = fmaf(scale[t], static_cast<float>(acc[t][i]), sum[t][i]);
                    }
                    to_go -= n;
                    k = 0;
                    ++tap;
                }
                if constexpr (RING > 0) wait_vmem<0>();   // (nothing arrives in the ring any more)
            }
            asm volatile("" : : "v"(touched));
            if (s0 + ns < (a.k + 63) >> 6) break;   // the sums go on with the next chunk (one phase: host)

            // ---- results of the phase --------------------------------------------------------------------------
            if constexpr (!INT_TAPS) {
                KernelArgs &a = args_again();
                const int lane = thread_again() & 63, l = lane & 31, h = lane >> 5;
                const Tables table = tables_of(a);
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
                // results of eight sums v of a pixel, channels ct .. ct + 7 (in the workgroup)
                auto scaled = [&](const float (&v)[8], const float *sw, const float *bias, Out (&res)[8]) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if constexpr (OUT == kOutI32) {
                            res[i] = static_cast<int>(v[i] * UNIT);   // (rounds towards zero)
                        } else {
                            // (scales of up to the largest float: they are not multiplied by the unit before their codes)
                            const float r = FOLD ? v[i] * UNIT : __builtin_rintf(v[i] * UNIT) * one_scale;
                            const float y = fmaf(r, sw[i], bias[i]);
                            if constexpr (OUT == kOutF16) res[i] = __float2half_rn(y);
                            else res[i] = y;
                        }
                    }
                };
                const uint32_t rows_left = min(a.pixels - p0, 128u << a.xw_log2);
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
                    float sw[16], bias[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        sw[i] = OUT != kOutI32 ? table.sw[ct + i] : 0.f;
                        bias[i] = OUT != kOutI32 ? table.bias[ct + i] : 0.f;
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
                            scaled(v, sw + 8 * half, bias + 8 * half, res[half]);
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
                        sw[i] = OUT != kOutI32 ? table.sw[ct + 8 * half0 + i] : 0.f;
                        bias[i] = OUT != kOutI32 ? table.bias[ct + 8 * half0 + i] : 0.f;
                    }
                    Out res[8];
                    scaled(v, sw, bias, res);
                    store8(res, px, c0 + 16 * h + 8 * half0);
                }
            }
            const int done = nw >> kl;
            first += done;
            left -= done;
            if (left == 0) return;
            shrink();
            if (RING && a.ring_shared) lds_barrier();   // nobody reads the exchange area any more
            begin_task(a);
        }

        // ---- next chunk -----------------------------------------------------------------------------------------
        s0 += ns;
        ns = min(a.chunk, ((a.k + 63) >> 6) - s0);
        KernelArgs &again = args_again();
        begin_fill(again);
        begin_task(again);
        lds_barrier();   // every wave is done with the resident steps
        clear_sums();
    }
}

}  // namespace

// One form's kernels by output type and weights' way (a file each, so that they compile in parallel); F16, F32, I32: those
// output types' rows, HQ_RESIDENT_WHOLE (of steps), HQ_RESIDENT_TAIL or HQ_RESIDENT_NONE.
#define HQ_RESIDENT_FORM(NAME, KIND, F16, F32, I32)                                                             \
    const void *NAME(int out, int form) {                                                                       \
        static const void *const kernels[3][7] = {F16(kOutF16, KIND), F32(kOutF32, KIND), I32(kOutI32, KIND)};  \
        return kernels[out == kOutF16 ? 0 : out == kOutF32 ? 1 : 2][form];                                      \
    }
#define HQ_RESIDENT_NONE(OUT, KIND) {}
#define HQ_RESIDENT_WHOLE(OUT, KIND) HQ_RESIDENT_ROW(OUT, KIND, false)
#define HQ_RESIDENT_TAIL(OUT, KIND) HQ_RESIDENT_ROW(OUT, KIND, true)
#define HQ_RESIDENT_ROW(OUT, KIND, TAIL)                                                                        \
    {HQ_RESIDENT_FN(OUT, KIND, 0, 0, TAIL), HQ_RESIDENT_FN(OUT, KIND, 0, 1, TAIL), HQ_RESIDENT_FN(OUT, KIND, 0, 2, TAIL), \
     HQ_RESIDENT_FN(OUT, KIND, 0, 3, TAIL), HQ_RESIDENT_FN(OUT, KIND, 0, 4, TAIL), HQ_RESIDENT_FN(OUT, KIND, 2, 0, TAIL), \
     HQ_RESIDENT_FN(OUT, KIND, 3, 0, TAIL)}
#define HQ_RESIDENT_FN(OUT, KIND, RING, NS, TAIL)                                                               \
    reinterpret_cast<const void *>(resident_kernel<OUT, KIND, RING, resident_unrolled(KIND, OUT, NS), TAIL>)
// form: the steps of an unrolled tap (1 .. 4), else 0 without a ring or 3 more than its slots
constexpr int resident_form(int ring, int ns) { return ns ? ns : ring ? ring + 3 : 0; }
