// nnp_split.hip -- the FP32 network GEMMs on the bf16 matrix cores, operands
// split into three bf16 parts (nnp_split.h).
#include "nnp_split.h"

namespace nnp {

// C = A B^T: A [rows][K] FP32 in memory, B pre-split in fragment order
// (split_index), both K-contiguous.  One workgroup owns a 16 FM x 16 FN WN
// tile, wave w the columns 16 FN w ..; K runs in 32-deep steps.
//
// The rows of a step are loaded as FP32 (32 bytes a thread), split in
// registers and written to one of two LDS stages as three bf16 tiles; the
// weight fragments go from L2 straight into registers, one step ahead.  Per
// step and wave at FM = FN = 4: 96 MFMAs (1536 clocks), 12 LDS fragment reads
// for the rows and 12 KiB of weight fragments; the split costs each thread
// about 44 vector instructions, which the other wave of the SIMD hides.
// Bound by the matrix cores: 33,248 ragged atoms, 8 ANI-2x models, forward
// 1146 -> 575 us and backward 1138 -> 642 us against the FP32 MFMA kernel
// (k_gemm, both operands through LDS), 1.46 / 1.31 PFLOP/s of bf16 products.
template <int FM, int FN, int WN, int EPI>
__global__ __launch_bounds__(64 * WN, 2) void k_gx(SplitArgs a) {
    constexpr int BM = 16 * FM, BN = 16 * FN * WN, NT = 64 * WN;
    constexpr int NTASK = BM * 4, NA = (NTASK + NT - 1) / NT;   // 8-value pieces of a row step per thread
    typedef bf16x8 Frag;
    __shared__ __align__(16) char lds[2][kParts * BM * 64];
    __shared__ float red[EPI == EPI_L3F ? BM * WN : 1];
    const GemmArgs<PrecF32>& g = a.g;

    // tile schedule as in k_gemm (XCD-contiguous ranges, kGroupM row tiles)
    const int T = g.nm * g.nn * g.nz;
    const int bid = blockIdx.x, xcd = bid & 7, slot = bid >> 3;
    const int q8 = T >> 3, r8 = T & 7;
    const int lin = xcd * q8 + (xcd < r8 ? xcd : r8) + slot;
    const int per_z = g.nm * g.nn;
    const int z = lin / per_z, rem = lin % per_z;
    const int grp = rem / (kGroupM * g.nn), inside = rem % (kGroupM * g.nn);
    const int gsz = min(kGroupM, g.nm - grp * kGroupM);
    const int tile_n = inside / gsz, tile_m = grp * kGroupM + inside % gsz;

    const int rows = g.info->rows;
    if (tile_m * BM >= rows) return;
    const int s = g.tile_species[(tile_m * BM) / g.row_tile];
    if (s < 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wn = __builtin_amdgcn_readfirstlane(tid >> 6);

    const float* A = g.A + (size_t)tile_m * BM * g.lda + (size_t)z * g.a_z;
    const int nk = g.K / 32;
    const bf16_t* Bw = a.Bx + (size_t)s * a.bx_s + (size_t)z * a.bx_z +
                       (size_t)(tile_n * (BN / 16) + wn * FN) * nk * (kParts * 512) + lane * 8;

    Frag bq[2][FN][kParts];
    auto load_b = [&](Frag(&b)[FN][kParts], int step) {
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int p = 0; p < kParts; ++p)
                b[j][p] = *(const Frag*)(Bw + ((size_t)(j * nk + step) * kParts + p) * 512);
    };
    float ar[2][NA][8];
    auto load_a = [&](float(&r)[NA][8], int step) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int t = tid + NT * u;
            if (NTASK % NT != 0 && t >= NTASK) continue;
            const float* p = A + (size_t)(t >> 2) * g.lda + step * 32 + (t & 3) * 8;
            *(float4*)&r[u][0] = *(const float4*)p;
            *(float4*)&r[u][4] = *(const float4*)(p + 4);
        }
    };
    auto store_a = [&](char* st, const float(&r)[NA][8]) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int t = tid + NT * u;
            if (NTASK % NT != 0 && t >= NTASK) continue;
            uint4 o[kParts];
            split8(r[u], o);
#pragma unroll
            for (int p = 0; p < kParts; ++p) *(uint4*)(st + split_at(BM, p, t >> 2, t & 3)) = o[p];
        }
    };
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;
    auto compute = [&](const char* st, const Frag(&b)[FN][kParts]) {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            Frag af[kParts];
#pragma unroll
            for (int p = 0; p < kParts; ++p)
                af[p] = *(const Frag*)(st + split_at(BM, p, i * 16 + (lane & 15), lane >> 4));
            split_mma(acc[i], b, af);
        }
    };

    load_a(ar[0], 0);
    load_b(bq[0], 0);
    load_a(ar[1], 1);   // K is a multiple of 64: at least two steps, an even number
    store_a(lds[0], ar[0]);
    __syncthreads();
    for (int kt = 0; kt < nk; kt += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int step = kt + u;
            load_b(bq[u ^ 1], min(step + 1, nk - 1));
            load_a(ar[u], min(step + 2, nk - 1));
            // the compiler would sink those loads towards their use
            asm volatile("" ::: "memory");
            compute(lds[u], bq[u]);
            store_a(lds[u ^ 1], ar[u ^ 1]);            // step + 1 (past the end: unread)
            __syncthreads();
        }
    }
    gemm_epilogue<PrecF32, EPI, BM, WN, FM, FN>(g, acc, lane, tile_m * BM, 0, tile_n * BN + wn * 16 * FN + 4 * (lane >> 4),
                                                s, z, wn, tile_n, red);
}

template <int FM, int FN, int WN, int EPI>
static hipError_t run_gx(SplitArgs a, int R, int N, hipStream_t st, const Timer& tm, const char* name) {
    constexpr int BM = 16 * FM, BN = 16 * FN * WN;
    a.g.nm = R / BM;
    a.g.nn = N / BN;
    if (a.g.K % 64 != 0 || a.g.K < 64 || N % BN != 0 || R % BM != 0 || a.g.row_tile % BM != 0 || !a.Bx)
        return hipErrorInvalidValue;
    tm.b(name, st);
    hipLaunchKernelGGL((k_gx<FM, FN, WN, EPI>), dim3(a.g.nm * a.g.nn * a.g.nz), dim3(64 * WN), 0, st, a);
    tm.e(name, st);
    return hipGetLastError();
}

template <int EPI>
hipError_t split_gemm(SplitArgs a, int R, int N, int nz, hipStream_t st, const Timer& tm, const char* name) {
    a.g.nz = nz;
    // layer 3's energy partials are counted per 64 columns
    if (EPI == EPI_L3F) return run_gx<4, 1, 4, EPI>(a, R, N, st, tm, name);
    if (N % 256 == 0) return run_gx<4, 4, 4, EPI>(a, R, N, st, tm, name);
    if (N % 192 == 0) return run_gx<4, 3, 4, EPI>(a, R, N, st, tm, name);
    if (N % 128 == 0) return run_gx<4, 2, 4, EPI>(a, R, N, st, tm, name);
    return run_gx<4, 1, 4, EPI>(a, R, N, st, tm, name);
}
#define NNP_SPLIT(EPI)                                                                                  \
    template hipError_t split_gemm<EPI>(SplitArgs, int, int, int, hipStream_t, const Timer&, const char*);
NNP_SPLIT(EPI_CELU)
NNP_SPLIT(EPI_L3F)
NNP_SPLIT(EPI_DSIG)
NNP_SPLIT(EPI_ACC)
NNP_SPLIT(EPI_RAW)
NNP_SPLIT(EPI_REV)

}  // namespace nnp
