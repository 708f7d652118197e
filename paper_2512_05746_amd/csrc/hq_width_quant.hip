// Activation side of the paper's own convolution (Method, "Convolution"): the NHWC tensor is
// read as rows of one image line each, X~ of shape (B C_in h) x w, transformed along the WIDTH
// axis with H_c = BlockDiag(H_k) and quantised with one scale for the whole tensor,
//     q = clamp(rne((X~ H_c) / S)).
// The integer convolution of that scheme runs on (X~ H_c)_int H_c,raw, i.e. on the codes taken
// back along the width axis with the +-1 matrix.  That integer product is formed here, in the
// same pass, exactly: u = q * BlockDiag(H_raw), |u| <= 2^(a_bits-1) * had_block <= 512, and stored
// as three signed base-16 digit planes, u = d0 + 16 d1 + 256 d2 with every digit in [-8, 7], each
// plane an NHWC tensor of packed nibbles.  The convolution then runs once per plane on the
// 4-bit path.
//
// One thread owns two neighbouring channels (one byte of packed digits per pixel and plane) of
// one transform block of one image line: it loads the 2 x had_block values, transforms them in
// registers (Sylvester order: the in-place butterfly with strides 1, 2, 4, ...), quantises,
// transforms the codes back in integers and writes the digits.  Neighbouring threads own
// neighbouring channel pairs, so loads and stores of a pixel are contiguous.
//
// What bounds it: instruction issue and the number of stores (12 bytes are moved per 4-byte load).  So both channels go
// back through one 32-bit butterfly (two 16-bit fields, |u| <= 512), the three digits of both come out of one addition
// (u + 0x888 holds digit + 8 in every nibble), and the bytes of four pixels are transposed over four lanes, which then
// store eight channels of one pixel each; a workgroup is as wide as the line's channels, so that no pass is nearly empty.
// 16 x 16 x 16 x 576, block 16: 15.0 -> 6.5 us (8.3 MB; the larger part is one wave's chain of load, transform and store).
#include <hip/hip_fp16.h>

#include <algorithm>

#include "hq_common.h"

namespace {

constexpr int kMaxThreads = 512;

__device__ __forceinline__ void load_pair(const __half *p, float &a, float &b) {
    const __half2 v = *reinterpret_cast<const __half2 *>(p);
    a = __low2float(v);
    b = __high2float(v);
}
__device__ __forceinline__ void load_pair(const float *p, float &a, float &b) {
    const float2 v = *reinterpret_cast<const float2 *>(p);
    a = v.x;
    b = v.y;
}

template <int B, typename V>
__device__ __forceinline__ void butterfly(V (&v)[B]) {
#pragma unroll
    for (int h = 1; h < B; h <<= 1)
#pragma unroll
        for (int i = 0; i < B; ++i)
            if ((i & h) == 0) {
                const V x = v[i], y = v[i + h];
                v[i] = x + y;
                v[i + h] = x - y;
            }
}

// Value of another lane of the quad (CTRL: quad_perm).
template <int CTRL>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, true));
}

// Byte i of lane j's dword <-> byte j of lane i's, over the four lanes of a quad.
__device__ __forceinline__ uint32_t transpose_quad(uint32_t v, uint32_t sel1, uint32_t sel2) {
    v = __builtin_amdgcn_perm(quad_lane<0xB1>(v), v, sel1);      // with lane ^ 1: bytes 0/2 <-> 1/3
    return __builtin_amdgcn_perm(quad_lane<0x4E>(v), v, sel2);   // with lane ^ 2: low <-> high half
}

// QUADS: c is a multiple of 8 and the block at least four pixels, so that quads of lanes are whole and their
// dwords aligned; otherwise every lane stores its own bytes.
template <typename T, int LOGB, bool QUADS>
__global__ __launch_bounds__(kMaxThreads) void width_quant_kernel(const T *__restrict__ x, int w, int c, float qmax,
                                                                  const float *__restrict__ given,
                                                                  uint8_t *__restrict__ xu3, uint32_t plane_bytes) {
    constexpr int B = 1 << LOGB;
    const int blocks_per_line = w >> LOGB;
    const uint32_t line = blockIdx.x / blocks_per_line;                     // image * h + row
    const uint32_t pix0 = line * w + (blockIdx.x % blocks_per_line) * B;   // first pixel of the block
    const int half_c = c >> 1;
    // the butterfly yields sqrt(B) x the orthonormal transform
    const float inv = 1.0f / (given[0] * sqrtf(static_cast<float>(B)));
    const int q = threadIdx.x & 3;
    const uint32_t sel1 = q & 1 ? 0x03070105u : 0x06020400u, sel2 = q & 2 ? 0x03020706u : 0x05040100u;
    for (int j = threadIdx.x; j < half_c; j += blockDim.x) {
        float v0[B], v1[B];
#pragma unroll
        for (int e = 0; e < B; ++e) load_pair(x + (static_cast<int64_t>(pix0 + e) * c + 2 * j), v0[e], v1[e]);
        butterfly<B>(v0);
        butterfly<B>(v1);
        int u[B];   // channel 2 j in the low half, 2 j + 1 in the high one
#pragma unroll
        for (int e = 0; e < B; ++e) {
            const int q0 = static_cast<int>(fminf(fmaxf(rintf(v0[e] * inv), -qmax - 1.0f), qmax));   // rint: ties to even
            const int q1 = static_cast<int>(fminf(fmaxf(rintf(v1[e] * inv), -qmax - 1.0f), qmax));
            u[e] = q0 + q1 * 65536;
        }
        butterfly<B>(u);
        uint32_t d[B];   // three digits of each half, two's complement
#pragma unroll
        for (int e = 0; e < B; ++e) d[e] = (static_cast<uint32_t>(u[e]) + 0x08880888u) ^ 0x08880888u;
        auto digits = [&](int e, int p) { return ((d[e] >> (4 * p)) & 15u) | ((d[e] >> (12 + 4 * p)) & 0xF0u); };
        if constexpr (QUADS) {
#pragma unroll
            for (int e = 0; e < B; e += 4) {
                uint8_t *dst = xu3 + (static_cast<int64_t>(pix0 + e + q) * half_c + (j & ~3));
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const uint32_t four = digits(e, p) | digits(e + 1, p) << 8 | digits(e + 2, p) << 16 | digits(e + 3, p) << 24;
                    *reinterpret_cast<uint32_t *>(dst + static_cast<int64_t>(p) * plane_bytes) = transpose_quad(four, sel1, sel2);
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < B; ++e) {
                uint8_t *dst = xu3 + (static_cast<int64_t>(pix0 + e) * half_c + j);
#pragma unroll
                for (int p = 0; p < 3; ++p) dst[static_cast<int64_t>(p) * plane_bytes] = static_cast<uint8_t>(digits(e, p));
            }
        }
    }
}

template <typename T>
hq_status launch_width_quant(const T *x, int64_t lines, int w, int c, int had_block, int bits, const float *given,
                             uint8_t *xu3, hipStream_t stream) {
    const hq::LaunchCheck check;   // samples the thread's error state before anything is launched
    const float qmax = static_cast<float>((1 << (bits - 1)) - 1);
    const int64_t grid = lines * (w / had_block);
    const int64_t plane = lines * w * (c / 2);
    if (grid > 0x7fffffffLL || lines * w > 0x7fffffffLL || plane > 0xffffffffLL) return HQ_ERR_SHAPE;
    const int pairs = std::min(c / 2, kMaxThreads);
    const dim3 g(static_cast<unsigned>(grid)), b((pairs + 63) & ~63);
    const bool quads = c % 8 == 0;
    const uint32_t pb = static_cast<uint32_t>(plane);
    switch (hq::ilog2(had_block)) {
#define HQ_WIDTH_CASE(L) \
    case L:                                                                                                             \
        if (L >= 2 && quads)                                                                                            \
            hipLaunchKernelGGL((width_quant_kernel<T, L, (L >= 2)>), g, b, 0, stream, x, w, c, qmax, given, xu3, pb);   \
        else                                                                                                            \
            hipLaunchKernelGGL((width_quant_kernel<T, L, false>), g, b, 0, stream, x, w, c, qmax, given, xu3, pb);      \
        break;
        HQ_WIDTH_CASE(0) HQ_WIDTH_CASE(1) HQ_WIDTH_CASE(2) HQ_WIDTH_CASE(3)
        HQ_WIDTH_CASE(4) HQ_WIDTH_CASE(5) HQ_WIDTH_CASE(6)
#undef HQ_WIDTH_CASE
        default: return HQ_ERR_SHAPE;
    }
    return check.status();
}

}  // namespace

extern "C" hq_status hq_act_hadamard_quant_width(const void *x, hq_dtype x_dtype, int nb, int h, int w, int c,
                                                 int had_block, int a_bits, const float *x_scale,
                                                 uint8_t *xu3, void *stream) {
    if (!x || !x_scale || !xu3) return HQ_ERR_NULL;
    if (x_dtype != HQ_F16 && x_dtype != HQ_F32) return HQ_ERR_DTYPE;
    if (a_bits < 2 || a_bits > 4) return HQ_ERR_BITS;
    if (nb <= 0 || h <= 0 || w <= 0 || c <= 0 || (c & 1)) return HQ_ERR_SHAPE;
    if (!hq::pow2_upto_128(had_block) || had_block > 64 || w % had_block != 0) return HQ_ERR_SHAPE;
    if (!hq::aligned16(x) || !hq::aligned16(xu3) || (reinterpret_cast<uintptr_t>(x_scale) & 3u)) return HQ_ERR_ALIGN;
    const int64_t lines = static_cast<int64_t>(nb) * h;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (x_dtype == HQ_F16)
        return launch_width_quant(static_cast<const __half *>(x), lines, w, c, had_block, a_bits, x_scale, xu3, s);
    return launch_width_quant(static_cast<const float *>(x), lines, w, c, had_block, a_bits, x_scale, xu3, s);
}
