// nnp_gemm.h -- pieces the network GEMM kernels share: MFMA operand types, the
// activation function, the kernels' arguments, row-vector access and the
// epilogues.
#pragma once

#include <algorithm>
#include <type_traits>

#include "nnp_internal.h"

namespace nnp {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));

template <typename TS> struct MF;
template <> struct MF<float> {
    static constexpr int KM = 4, KL = 1;   // K of one MFMA, K elements per lane
    typedef float Frag;
    typedef f32x4 Acc;
    __device__ static Acc mma(Frag a, Frag b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // with the operands swapped (B fragment first) accumulator element r of
    // lane l holds C[l % 16][col0(l) + r * kColStride]
    static constexpr int kColStride = 1;
    __device__ static int col0(int l) { return 4 * (l >> 4); }
};
template <> struct MF<double> {
    static constexpr int KM = 4, KL = 1;
    typedef double Frag;
    typedef f64x4 Acc;
    __device__ static Acc mma(Frag a, Frag b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // the FP64 16x16x4 accumulator interleaves its rows across the lane
    // groups, so a lane's four elements are every fourth column
    static constexpr int kColStride = 4;
    __device__ static int col0(int l) { return l >> 4; }
};
template <> struct MF<bf16_t> {
    static constexpr int KM = 32, KL = 8;
    typedef bf16x8 Frag;
    typedef f32x4 Acc;
    __device__ static Acc mma(Frag a, Frag b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    static constexpr int kColStride = 1;
    __device__ static int col0(int l) { return 4 * (l >> 4); }
};

enum { EPI_CELU = 0, EPI_L3F = 1, EPI_DSIG = 2, EPI_ACC = 3, EPI_RAW = 4, EPI_REV = 5 };

// CELU and its derivative, branch-free (the exponential is taken of min(z, 0)
// and always finite); ial = 1 / alpha.  CELU'(z) is recovered from a stored
// h = CELU(z): h >= 0 <=> z >= 0, and exp(z / alpha) = 1 + h / alpha.
// (float: the scaled argument is clamped, min(z c, 0) = min(z, 0) c for c > 0,
// so the minimum takes a product and needs no NaN canonicalisation of z)
__device__ inline float celu(float z, float al, float ial) {
    const float e = __builtin_amdgcn_exp2f(fminf(z * (ial * 1.44269504088896341f), 0.f));
    return z >= 0.f ? z : __builtin_fmaf(al, e, -al);
}
__device__ inline double celu(double z, double al, double ial) {
    const double e = expm1(fmin(z, 0.0) * ial);
    return z >= 0.0 ? z : al * e;
}
__device__ inline float dcelu_z(float z, float ial) {
    // exp2 of the clamped argument is exactly 1 for z >= 0
    return __builtin_amdgcn_exp2f(fminf(z * (ial * 1.44269504088896341f), 0.f));
}
__device__ inline double dcelu_z(double z, double ial) {
    const double e = exp(fmin(z, 0.0) * ial);
    return z >= 0.0 ? 1.0 : e;
}
// (1 + h / alpha >= 1 exactly when h >= 0, so the minimum selects the branch)
__device__ inline float dcelu_h(float h, float ial) { return fminf(__builtin_fmaf(h, ial, 1.f), 1.f); }
__device__ inline double dcelu_h(double h, double ial) { return h >= 0.0 ? 1.0 : 1.0 + h * ial; }

template <typename P> struct GemmArgs {
    typedef typename P::TS TS;
    typedef typename P::TA TA;
    const TS* A; int lda; long a_z;
    const TS* B; int ldb; long b_s, b_z;
    const TA* bias; long bias_s, bias_z;
    void* C; int ldc; long c_z;
    const TS* Hr; int ldh; long h_z;        // stored activations for CELU'
    void* C2; long c2_z;                     // second output (EPI_REV), leading dim ldc
    const TS* X; int ldx; long x_z;          // auxiliary product (EPI_REV)
    const TS* Tr; int ldt; long t_z;         // tangent activations (EPI_REV)
    const TA* w4; long w4_s, w4_z;
    TA* epart; int n_models, nt;
    TA gscale, alpha, inv_alpha;
    int K;
    const int32_t* tile_species; int row_tile;
    const BucketInfo* info;
    int nm, nn, nz;                          // tiles along M (launch bound), N and models
    int pick_rows;                           // rows that the choice of a K split goes by
};

// Four output elements of one row held by one lane: columns c, c+ST, c+2ST,
// c+3ST (ST = 1 for the f32 / bf16 MFMAs, 4 for f64).
template <typename TS, int ST> struct Quad {
    typedef typename std::conditional<sizeof(TS) == 8, double, float>::type TA;
    __device__ static void ld(const TS* p, TA v[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = Store<TS>::ld(p[r * ST]);
    }
    __device__ static void st(TS* p, const TA v[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r * ST] = Store<TS>::st(v[r]);
    }
};
template <> struct Quad<float, 1> {
    __device__ static void ld(const float* p, float v[4]) {
        const float4 q = *(const float4*)p;
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    }
    __device__ static void st(float* p, const float v[4]) { *(float4*)p = make_float4(v[0], v[1], v[2], v[3]); }
};
template <> struct Quad<bf16_t, 1> {
    __device__ static void ld(const bf16_t* p, float v[4]) {
        const uint2 q = *(const uint2*)p;
        v[0] = bf2f((bf16_t)(q.x & 0xffffu)); v[1] = bf2f((bf16_t)(q.x >> 16));
        v[2] = bf2f((bf16_t)(q.y & 0xffffu)); v[3] = bf2f((bf16_t)(q.y >> 16));
    }
    __device__ static void st(bf16_t* p, const float v[4]) {
        uint2 q;
        q.x = pack_bf16x2(v[0], v[1]);
        q.y = pack_bf16x2(v[2], v[3]);
        *(uint2*)p = q;
    }
};

// This workgroup's tile among the T in use (at most the grid), or -1.  Block
// ids are dealt round-robin to the 8 XCDs; XCD x gets the contiguous range of
// tiles it would own in order.
__device__ inline int xcd_tile(int T) {
    const int bid = blockIdx.x, xcd = bid & 7, slot = bid >> 3;
    const int q8 = T >> 3, r8 = T & 7;
    if (slot >= q8 + (xcd < r8 ? 1 : 0)) return -1;
    return xcd * q8 + (xcd < r8 ? xcd : r8) + slot;
}
// Row tiles the schedule deals out: those the buckets hold, known on the
// device only, so that every XCD's range is as long (48 molecules in a
// 128-molecule handle: layer 1 56 -> 33 us); for 16-row tiles the launch's
// bound, which is at most 7 tiles more and spares small calls the wait for
// that count before the index arithmetic (about 0.6 us a kernel).
template <int BM> __device__ inline int row_tiles(const BucketInfo* info, int bound) {
    if constexpr (BM == 16) return bound;
    else return info->rows / BM;
}

// Row tiles are grouped kGroupM at a time: within a group the schedule runs
// M-fastest, so the tiles an XCD has in flight share both a few row blocks
// and a few weight column blocks in its L2.
constexpr int kGroupM = 8;

// the fused tails are compiled for the ANI-2x hidden widths (256, 192, 160
// padded to 192); other widths take the per-layer GEMMs
constexpr int kTailH1 = 256, kTailH2 = 192, kTailH3 = 192;

// Epilogue of one wave's FM x FN MFMA tiles of the product C = A B^T: element r
// of acc[i][j] in lane l is C[row_base + lrow0 + 16 i + l % 16][col0 + 16 j +
// r ST], col0 = the wave's first column + col0(l).  s: element, z: model,
// red: LDS [BM][WN] (layer 3 only), wn: this wave's place among the WN that
// share its rows.
template <typename P, int EPI, int BM, int WN, int FM, int FN>
__device__ inline void gemm_epilogue(const GemmArgs<P>& g, const typename MF<typename P::TS>::Acc (&acc)[FM][FN],
                                     int lane, int row_base, int lrow0, int col0, int s, int z, int wn,
                                     int tile_n, typename P::TA* red) {
    typedef typename P::TS TS;
    typedef typename P::TA TA;
    constexpr int ST = MF<TS>::kColStride;
    typedef Quad<TS, ST> Q;
    const int row0 = row_base + lrow0 + (lane & 15);

    if (EPI == EPI_CELU) {
        TS* C = (TS*)g.C + (size_t)z * g.c_z;
        const TA* bias = g.bias + (size_t)s * g.bias_s + (size_t)z * g.bias_z;
        TA bb[FN][4];   // all requested before the first store
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) bb[j][r] = bias[col0 + j * 16 + r * ST];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = col0 + j * 16;
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                TA v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = celu((TA)acc[i][j][r] + bb[j][r], g.alpha, g.inv_alpha);
                Q::st(C + (size_t)(row0 + i * 16) * g.ldc + col, v);
            }
        }
    } else if (EPI == EPI_ACC) {
        // dE/dAEV rows, in the precision's dE/dAEV storage type
        typedef typename P::TG TG;
        TG* C = (TG*)g.C + (size_t)z * g.c_z;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                TA v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (TA)acc[i][j][r];
                Quad<TG, ST>::st(C + (size_t)(row0 + i * 16) * g.ldc + col0 + j * 16, v);
            }
    } else if (EPI == EPI_DSIG) {
        TS* C = (TS*)g.C + (size_t)z * g.c_z;
        const TS* Hr = g.Hr + (size_t)z * g.h_z;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const size_t row = row0 + i * 16;
                const int col = col0 + j * 16;
                TA hh[4], v[4];
                Q::ld(Hr + row * g.ldh + col, hh);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (TA)acc[i][j][r] * dcelu_h(hh[r], g.inv_alpha);
                Q::st(C + row * g.ldc + col, v);
            }
    } else if (EPI == EPI_RAW) {
        TS* C = (TS*)g.C + (size_t)z * g.c_z;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                TA v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (TA)acc[i][j][r];
                Q::st(C + (size_t)(row0 + i * 16) * g.ldc + col0 + j * 16, v);
            }
    } else if (EPI == EPI_REV) {
        // reverse step through h = CELU(z) and its tangent hdot = CELU'(z) zdot:
        //   zbar    = abar CELU'(z) + acheck (CELU''/CELU')(z) hdot
        //   zdotbar = acheck CELU'(z)
        // abar = this product, acheck = X (the same product of the tangent
        // adjoint), CELU''/CELU' = 1/alpha for z < 0 and 0 otherwise.
        TS* C = (TS*)g.C + (size_t)z * g.c_z;
        TS* C2 = (TS*)g.C2 + (size_t)z * g.c2_z;
        const TS* Hr = g.Hr + (size_t)z * g.h_z;
        const TS* X = g.X + (size_t)z * g.x_z;
        const TS* Tr = g.Tr + (size_t)z * g.t_z;
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                const size_t row = row0 + i * 16;
                const int col = col0 + j * 16;
                TA hh[4], ac[4], hd[4], v[4], v2[4];
                Q::ld(Hr + row * g.ldh + col, hh);
                Q::ld(X + row * g.ldx + col, ac);
                Q::ld(Tr + row * g.ldt + col, hd);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const TA d1 = dcelu_h(hh[r], g.inv_alpha);
                    const TA rho = hh[r] < TA(0) ? g.inv_alpha : TA(0);
                    v[r] = (TA)acc[i][j][r] * d1 + ac[r] * rho * hd[r];
                    v2[r] = ac[r] * d1;
                }
                Q::st(C + row * g.ldc + col, v);
                Q::st(C2 + row * g.ldc + col, v2);
            }
    } else {   // EPI_L3F
        TS* C = (TS*)g.C + (size_t)z * g.c_z;
        const TA* bias = g.bias + (size_t)s * g.bias_s + (size_t)z * g.bias_z;
        const TA* w4 = g.w4 + (size_t)s * g.w4_s + (size_t)z * g.w4_z;
        TA part[FM];
#pragma unroll
        for (int i = 0; i < FM; ++i) part[i] = 0;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int col = col0 + j * 16;
            TA bb[4], ww[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                bb[r] = bias[col + r * ST];
                ww[r] = w4[col + r * ST];
            }
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                TA v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const TA zz = (TA)acc[i][j][r] + bb[r];
                    part[i] += ww[r] * celu(zz, g.alpha, g.inv_alpha);
                    v[r] = dcelu_z(zz, g.inv_alpha) * ww[r] * g.gscale;
                }
                Q::st(C + (size_t)(row0 + i * 16) * g.ldc + col, v);
            }
        }
        // sum over the four lane groups (same row, different columns), then
        // over the WN waves that share the row
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            TA v = part[i];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (lane < 16) red[(lrow0 + i * 16 + lane) * WN + wn] = v;
        }
        __syncthreads();
        for (int rr = threadIdx.x; rr < BM; rr += blockDim.x) {
            TA v = 0;
#pragma unroll
            for (int q = 0; q < WN; ++q) v += red[rr * WN + q];
            const size_t row = (size_t)row_base + rr;
            g.epart[(row * g.n_models + z) * g.nt + tile_n] = v;
        }
    }
}

}  // namespace nnp
