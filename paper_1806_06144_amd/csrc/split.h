// Split-precision operands of the 16-bit matrix cores, shared by the packing
// kernels and the fused passes that read them.
//
// Feature rows. A float32 row x is scaled by a power of two so that its
// largest element lies in [2^14, 2^15) and stored as two fp16 planes, hi =
// fp16(x), lo = fp16(x - hi). hi + lo is x to 2^-23 of an element, and to
// 2^-39 of the row's largest element for those below 2^-16 of it. What is
// computed is the distance between packed rows: their norms are summed (in
// float64) from hi + lo, so rows that share values, however large, are not
// moved apart by their rounding.
//
// The dot product is formed as lo.hi + hi.lo + hi.hi (exact products, float32
// accumulation). The fourth term moves a squared distance by 2 lo_x.lo_z, at
// most |lo_x|^2 + |lo_z|^2. For most rows |lo|^2 is 0.6 to 0.7 of 2^-24 |x|^2,
// about the rounding of the norms themselves, but a row dominated by a few
// values that lie badly between fp16 numbers has up to 2^-22, and rows that
// share them are all moved alike. Panels of centres with a row above kLoLoMax
// are therefore multiplied with the fourth product too.
//
// Errors against float64 with float32 operands, with three products and norms
// of the unpacked rows, and as above: squared distances of 16 normal features
// beside a constant column of 64.03, root mean square in units of 2^-24 of the
// norms, 2.3 (0.9 with the column last), 8.6, 2.0; 64 features with it 4.2,
// 8.8, 2.7; 784 with it 11.4, 10.1, 7.0; 784 normal features 1.34, 1.31, 1.31;
// 784 uniform 5.3, 3.3, 3.3 (an instruction takes 32 features, so the
// accumulator is rounded d / 32 times, not d / 2). Rows of few features show
// the packing: 12 of 784 features 0.61, 0.61, 0.83. Sums over 20000 to 43000
// centres, relative: 16 features and the column 7.3e-5, 2.6e-4, 6.7e-5;
// without it 4.1e-7, 1.8e-7, 1.9e-7; 12 of 784 features 4.8e-7, 2.1e-7, 2.1e-7.
//
// A row that holds an infinity is stored as its infinite elements alone, +-1,
// with an infinite norm and inverse scale: its distances come out infinite
// where the dot product is negative and NaN (taken as 0) elsewhere, as those
// of float32 operands do. NaN elements make the norm NaN.
//
// Weights and kernel values (no common scale: both may span the whole
// float32 range) are stored as three bf16 planes, hi + mid + lo, which
// represent a float32 exactly; of the nine products the six largest are
// formed and the dropped ones are below 2^-26 of the product.
//
// All planes are laid out as operands of v_mfma_f32_16x16x32: a fragment of
// 16 rows x 32 depth is 1 KB, lane l holding row l % 16 and depth 8 (l / 16)
// .. + 7 in 16 contiguous bytes, so a wave's operand load is one contiguous
// kilobyte, from global memory, into LDS (in the order lane x 16 bytes that
// direct-to-LDS loads write) and out of it without bank conflicts.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ep {

constexpr int kFragBytes = 1024;      // one 16 x 32 operand plane
constexpr int kCPanel = 128;          // centre rows per packed panel
constexpr int kQPanel = 64;           // query rows per packed panel

// Bound of |lo|^2 / |x|^2 up to which lo.lo is left out: with both rows below
// it, it is at most 2^-24 of the norms.
constexpr double kLoLoMax = 1.0 / (1 << 24);

// 32-deep feature steps of a row of d features.
inline __host__ __device__ int64_t feature_steps(int64_t d) { return (d + 31) / 32; }
// Bytes of a panel of P rows: two planes, then P norms and P inverse scales.
inline __host__ __device__ int64_t panel_bytes(int64_t P, int64_t d) {
    return feature_steps(d) * (P / 16) * 2 * kFragBytes + P * 8;
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma_f16(uintx4 a, uintx4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a),
                                                  __builtin_bit_cast(half8, b), c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma_bf16(uintx4 a, uintx4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    const floatx2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf16_lo(unsigned u) { return __builtin_bit_cast(float, u << 16); }
__device__ __forceinline__ float bf16_hi(unsigned u) {
    return __builtin_bit_cast(float, u & 0xffff0000u);
}
// Two finite values as three bf16 pairs (a in the low halves).
__device__ __forceinline__ void split3(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
    h = pack_bf16(a, b);
    a -= bf16_lo(h);
    b -= bf16_hi(h);
    m = pack_bf16(a, b);
    a -= bf16_lo(m);
    b -= bf16_hi(m);
    l = pack_bf16(a, b);
}

// Where the weight of (centre c, label j) lies in the planes of a weight
// matrix with lt label tiles of 16: element index of plane 0 (bf16 units;
// planes are 512 elements apart). In a 32-centre group, lane group g = lane
// / 16 of the fragment holds the centres 16 (e / 4) + 4 g + e % 4, e = 0..7:
// the order in which a lane's accumulators of the distance product hold them.
__device__ __forceinline__ int64_t weight_elem(int64_t c, int64_t j, int64_t lt) {
    const int64_t group = c >> 5;
    const int r = (int)(c & 31);
    const int g = (r >> 2) & 3;
    const int e = ((r >> 4) << 2) | (r & 3);
    return ((group * lt + (j >> 4)) * 3 * 64 + (int64_t)(g * 16 + (int)(j & 15))) * 8 + e;
}
inline __host__ __device__ int64_t weight_plane_bytes(int64_t n_pad, int64_t lt) {
    return (n_pad / 32) * lt * 3 * kFragBytes;
}
// The three planes of one weight. Values that round up to infinity in bf16
// keep their largest finite head. Infinities and NaN go into the low plane,
// which meets only the heads of kernel values: a head times infinity is
// infinite, as in float32, where a zero mid or low plane would make it NaN.
__device__ __forceinline__ void split_weight(float w, unsigned short& hi, unsigned short& mid,
                                             unsigned short& lo) {
    unsigned h = 0, m = 0, l = 0;
    if (__builtin_isfinite(w)) {
        h = pack_bf16(w, 0.f) & 0xffffu;
        if ((h & 0x7fffu) == 0x7f80u) h -= 1;
        float r = w - bf16_lo(h);
        m = pack_bf16(r, 0.f) & 0xffffu;
        r -= bf16_lo(m);
        l = pack_bf16(r, 0.f) & 0xffffu;
    } else {
        l = pack_bf16(w, 0.f) & 0xffffu;
    }
    hi = (unsigned short)h;
    mid = (unsigned short)m;
    lo = (unsigned short)l;
}
__device__ __forceinline__ void store_weight(unsigned short* planes, int64_t at, float w) {
    split_weight(w, planes[at], planes[at + 512], planes[at + 1024]);
}

}  // namespace ep
