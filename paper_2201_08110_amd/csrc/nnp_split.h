// nnp_split.h -- FP32 operands as three bf16 parts for the bf16 matrix cores.
//
// x = h + m + l with h the bf16 of x's leading bits, m = bf16(x - h) and l =
// bf16(x - h - m) rounded to nearest: |m| <= 2^-7 |x|, |l| <= 2^-16 |x|, and the
// three hold every bit of the FP32 significand (short of underflow below
// 2^-110).  A product x y is formed as the six parts of weight >= 2^-16,
//   l h' + h l' + m m' + m h' + h m' + h h',
// each exact in FP32; the three dropped ones are at most 2^-22 of |x y|, 2^-25
// on average over the products of a sum (a sum of 1,024 with its FP32 additions:
// 2.5e-7 of its size, 3.2 to 5.7e-7 in a chain of fused multiply-adds).  gfx950
// runs bf16 MFMAs 16 times as fast as FP32 ones, so six of them take 0.375 of
// the FP32 MFMA's time.
// h is cut, not rounded: the nearest bf16 of a finite x above 3.39e38 is
// infinite.  An infinite or NaN x gives a part that is NaN, so a product that is.
#pragma once

#include "nnp_gemm.h"

namespace nnp {

constexpr int kParts = 3;
constexpr int kSplitRows = 64;   // bucket row tile of the handles that split their operands

// parts of two values, packed (low half = first)
__device__ inline void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);   // upper halves of both
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    m = pack_bf16x2(ra, rb);
    const float sa = ra - __uint_as_float(m << 16), sb = rb - __uint_as_float(m & 0xffff0000u);
    l = pack_bf16x2(sa, sb);
}
// eight values as one 16-byte chunk (or fragment) per part
__device__ inline void split8(const float v[8], uint4 o[kParts]) {
    split2(v[0], v[1], o[0].x, o[1].x, o[2].x);
    split2(v[2], v[3], o[0].y, o[1].y, o[2].y);
    split2(v[4], v[5], o[0].z, o[1].z, o[2].z);
    split2(v[6], v[7], o[0].w, o[1].w, o[2].w);
}

__device__ inline void split8(const float v[8], bf16x8 (&f)[kParts]) {
    uint4 o[kParts];
    split8(v, o);
#pragma unroll
    for (int p = 0; p < kParts; ++p) f[p] = __builtin_bit_cast(bf16x8, o[p]);
}

// LDS tile of split operands for one 32-deep k-step: [part][rows][64 bytes],
// the four 16-byte chunks of row r at position c ^ (r / 2 % 4): the eight
// rows a 16-byte read or write touches at a time then lie in distinct banks
__device__ inline int split_at(int rows, int part, int r, int c) {
    return (part * rows + r) * 64 + ((c ^ (r >> 1)) & 3) * 16;
}

// acc[j] += a b[j], smallest products first, the accumulators in turn
template <int FN>
__device__ inline void split_mma(f32x4 (&acc)[FN], const bf16x8 (&b)[FN][kParts], const bf16x8 (&a)[kParts]) {
    constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[j] = MF<bf16_t>::mma(b[j][pb[q]], a[pa[q]], acc[j]);
}

// arguments of a split GEMM: g.B is the FP32 weight operand in fragment order
// (frag_index), Bx its parts (split_index; bx_s / bx_z bf16 elements apart per
// element and model), null on handles with 16-row buckets
struct SplitArgs {
    GemmArgs<PrecF32> g;
    const bf16_t* Bx;
    long bx_s, bx_z;
};
// C = A B^T for R rows (a multiple of the bucket row tile), N columns, nz models
template <int EPI>
hipError_t split_gemm(SplitArgs a, int R, int N, int nz, hipStream_t st, const Timer& tm, const char* name);

// layers 2-3 forward and backward (widths of mlp_fused_supported)
hipError_t split_tail(const Shape& sh, const DevWeights<PrecF32>& wt, Work<PrecF32>& w, hipStream_t st, const Timer& tm);

}  // namespace nnp
