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
// step and wave at FM = 4, FN = 2: 48 MFMAs (768 clocks), 12 LDS fragment
// reads for the rows and 6 KiB of weight fragments; the split costs each
// thread about 44 vector instructions, which the other waves of the SIMD hide.
// Bound by the matrix cores: 33,248 ragged atoms, 8 ANI-2x models, forward
// 1146 -> 550 us and backward 1138 -> 600 us against the FP32 MFMA kernel
// (k_gemm, both operands through LDS), about 1.5 / 1.4 PFLOP/s of bf16 products.
template <int FM, int FN, int WN, int EPI>
__global__ __launch_bounds__(64 * WN, 2) void k_gx(SplitArgs a) {
    constexpr int BM = 16 * FM, BN = 16 * FN * WN, NT = 64 * WN;
    constexpr int NTASK = BM * 4, NA = (NTASK + NT - 1) / NT;   // 8-value pieces of a row step per thread
    typedef bf16x8 Frag;
    __shared__ __align__(16) char lds[2][kParts * BM * 64];
    __shared__ float red[EPI == EPI_L3F ? BM * WN : 1];
    const GemmArgs<PrecF32>& g = a.g;

    // tile schedule as in k_gemm (XCD-contiguous ranges, kGroupM row tiles)
    const int nm = g.info->rows / BM, per_z = nm * g.nn;
    const int lin = xcd_tile(per_z * g.nz);
    if (lin < 0) return;
    const int z = lin / per_z, rem = lin % per_z;
    const int grp = rem / (kGroupM * g.nn), inside = rem % (kGroupM * g.nn);
    const int gsz = min(kGroupM, nm - grp * kGroupM);
    const int tile_n = inside / gsz, tile_m = grp * kGroupM + inside % gsz;

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

// The same product where there are few tiles (or 16-row buckets): the eight
// waves of a workgroup split K instead of the columns, so a 16 FM x 64 tile's
// chain is an eighth as long and needs no barrier.  Both operands are FP32 in
// memory (weights in fragment order, a third fewer bytes than their parts: few
// rows are bound by reading the weights once), loaded straight into registers
// and split there; within a step lane group g holds k = 4 g + 0..3 and
// 16 + 4 g + 0..3 of both operands.  A wave takes U steps a round, all
// requested before the first is used, each buffer again as soon as it is
// split; steps past its share multiply zeros.  The waves' sums meet in LDS,
// each wave finishing its share of the 16 x 16 pieces.
template <int FM, int FN, int KW> struct KSplit {
    static constexpr int TN = FM * FN;               // pieces of the tile
    static constexpr int TW = (TN + KW - 1) / KW;    // pieces a wave finishes
    static constexpr size_t part = (size_t)KW * TN * 64 * 16;
    static constexpr size_t lds_bytes = part + sizeof(float) * 16 * FM * (FN / TW);
};

template <int FM, int FN, int KW, int U, int EPI>
__global__ __launch_bounds__(64 * KW, 2) void k_gxk(SplitArgs a) {
    touch_kernargs<sizeof(SplitArgs)>();
    typedef KSplit<FM, FN, KW> Ks;
    constexpr int TN = Ks::TN, TW = Ks::TW, BM = 16 * FM, BN = 16 * FN;
    extern __shared__ __align__(16) char smem[];
    const GemmArgs<PrecF32>& g = a.g;
    const int nm = row_tiles<BM>(g.info, g.nm), per_z = nm * g.nn;
    const int lin = xcd_tile(per_z * g.nz);
    if (lin < 0) return;
    const int z = lin / per_z, rem = lin % per_z;
    const int tile_n = rem / nm, tile_m = rem % nm;   // M-fastest: the weights are read once
    if (tile_m * BM >= g.info->rows) return;
    const int s = g.tile_species[(tile_m * BM) / g.row_tile];
    if (s < 0) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nk = g.K / 32, rounds = (nk + KW * U - 1) / (KW * U), k0 = wave * rounds * U;

    const float* Ap = g.A + (size_t)(tile_m * BM + (lane & 15)) * g.lda + (size_t)z * g.a_z + 4 * (lane >> 4);
    const float* Bp = g.B + (size_t)s * g.b_s + (size_t)z * g.b_z + (size_t)tile_n * FN * nk * 512 + lane * 4;
    float av[U][FM][8], bv[U][FN][8];
    auto load = [&](int u, int step) {
        const int st = min(step, nk - 1);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const float* p = Bp + (size_t)(j * nk + st) * 512;
            *(float4*)&bv[u][j][0] = *(const float4*)p;
            *(float4*)&bv[u][j][4] = *(const float4*)(p + 256);
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const float* p = Ap + (size_t)i * 16 * g.lda + st * 32;
            *(float4*)&av[u][i][0] = *(const float4*)p;
            *(float4*)&av[u][i][4] = *(const float4*)(p + 16);
        }
    };
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;
    auto round = [&](int kb, auto more) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bf16x8 bq[FN][kParts], aq[FM][kParts];
#pragma unroll
            for (int j = 0; j < FN; ++j) split8(bv[u][j], bq[j]);
            if (kb + u >= nk)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) av[u][i][e] = 0.f;
#pragma unroll
            for (int i = 0; i < FM; ++i) split8(av[u][i], aq[i]);
            if constexpr (more.value) {
                load(u, kb + u + U);
                asm volatile("" ::: "memory");   // the loads stay ahead of the products
            }
#pragma unroll
            for (int i = 0; i < FM; ++i) split_mma(acc[i], bq, aq[i]);
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load(u, k0 + u);
    for (int r = 0; r < rounds - 1; ++r) round(k0 + r * U, std::true_type{});
    round(k0 + (rounds - 1) * U, std::false_type{});
    f32x4* part = (f32x4*)smem;                        // [wave][piece][lane]
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) part[(size_t)(wave * TN + i * FN + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    // fewer pieces than waves: the others are done, or, where the epilogue has
    // a barrier, finish a piece a second time (the same values)
    if (EPI != EPI_L3F && wave * TW >= TN) return;
    const int t0 = wave * TW % TN;
    f32x4 sum[1][TW];
#pragma unroll
    for (int t = 0; t < TW; ++t) {
        sum[0][t] = part[(size_t)(t0 + t) * 64 + lane];
#pragma unroll
        for (int w = 1; w < KW; ++w) sum[0][t] += part[(size_t)(w * TN + t0 + t) * 64 + lane];
    }
    gemm_epilogue<PrecF32, EPI, BM, FN / TW, 1, TW>(g, sum, lane, tile_m * BM, 16 * (t0 / FN),
                                                    tile_n * BN + 16 * (t0 % FN) + 4 * (lane >> 4), s, z, t0 % FN / TW,
                                                    tile_n, (float*)(smem + Ks::part));
}

template <int FM, int FN, int KW, int U, int EPI>
static hipError_t run_gxk(SplitArgs a, int R, int N, hipStream_t st, const Timer& tm, const char* name) {
    typedef KSplit<FM, FN, KW> Ks;
    constexpr int BM = 16 * FM, BN = 16 * FN;
    a.g.nm = R / BM;
    a.g.nn = N / BN;
    if (a.g.K % 32 != 0 || a.g.K < 32 || N % BN != 0 || R % BM != 0 || a.g.row_tile % BM != 0 || !a.g.B)
        return hipErrorInvalidValue;
    auto kern = k_gxk<FM, FN, KW, U, EPI>;
    hipError_t e = ensure_lds((const void*)kern, Ks::lds_bytes);
    if (e != hipSuccess) return e;
    tm.b(name, st);
    hipLaunchKernelGGL(kern, dim3(a.g.nm * a.g.nn * a.g.nz), dim3(64 * KW), Ks::lds_bytes, st, a);
    tm.e(name, st);
    return hipGetLastError();
}

template <int FM, int FN, int WN, int EPI>
static hipError_t run_gx(SplitArgs a, int R, int N, hipStream_t st, const Timer& tm, const char* name) {
    constexpr int BM = 16 * FM, BN = 16 * FN * WN;
    a.g.nn = N / BN;
    if (a.g.K % 64 != 0 || a.g.K < 64 || N % BN != 0 || R % BM != 0 || a.g.row_tile % BM != 0 || !a.Bx)
        return hipErrorInvalidValue;
    tm.b(name, st);
    hipLaunchKernelGGL((k_gx<FM, FN, WN, EPI>), dim3(R / BM * a.g.nn * a.g.nz), dim3(64 * WN), 0, st, a);
    tm.e(name, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The fused tail (layers 2 and 3 forward, output layer, and the backward
// through them down to DZ1) for one row tile and model, as k_tail runs it but
// with split operands.  Every activation lives in LDS as three bf16 parts, one
// [part][BM][64-byte] tile per 32 columns (split_at); CELU' is taken from the
// parts' sum, which is the FP32 value itself.  32 rows and four waves, each a
// column quarter: 70 KB of LDS, two workgroups per CU, so one's epilogues and
// barriers run under the other's products (64 rows on eight waves, one
// workgroup per CU: 577 against 476 us on 33,248 ragged atoms, 37 against
// 26 us on 570).  Bound by the weight fragments' bytes from L2, one 16-byte
// lane load per two MFMAs.  The FP32 MFMA tail (k_tail) took 774 and 53 us.
template <int H1, int H2, int H3, int BM> struct SplitTail {
    static constexpr int tile = kParts * BM * 64;                  // one 32-column step
    static constexpr int h1 = H1 / 32 * tile, h2 = H2 / 32 * tile, h3 = H3 / 32 * tile;
    // H1 spans H2 / DZ2 and DZ3: it is dead once the first product is done
    static constexpr int acts = h1 > h2 + h3 ? h1 : h2 + h3;
    static constexpr int par = 4 * (H2 + 2 * H3), red = 4 * BM * 4;
    static constexpr int lds_bytes = acts + par + red;
};

struct SplitTailArgs {
    const float* H1;
    float* DZ1;
    int ldh;                                    // [Rcap][M*H1]
    const bf16_t *W2x, *W2Tx, *W3x, *W3Tx;      // split, fragment order
    const float *b2, *b3, *w4;
    float* epart;                               // [Rcap][M]
    float gscale, alpha, inv_alpha;
    int M, H3s;                                 // models; stored width of layer 3
    const int32_t* tile_species;
    int row_tile;
    const BucketInfo* info;
};

// acc = A rows [0, 16 FM) (LDS step tiles of BM rows) x B^T over K, B
// n-tiles nt0 + [0, FN) of a split matrix stored with KS / 32 steps per
// n-tile; its fragments are requested one step ahead.  bias: this lane's
// columns' starting values, or null.
template <int BM, int FM, int FN, int K, int KS>
__device__ inline void split_product(f32x4 (&acc)[FM][FN], const char* As, const bf16_t* __restrict__ Bx,
                                     int nt0, int lane, const float* bias) {
    typedef bf16x8 Frag;
    constexpr int NS = K / 32, NSS = KS / 32;
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float b0 = bias ? bias[j * 16 + r] : 0.f;
#pragma unroll
            for (int i = 0; i < FM; ++i) acc[i][j][r] = b0;
        }
    const bf16_t* Bl = Bx + (size_t)nt0 * NSS * (kParts * 512) + lane * 8;
    Frag bq[2][FN][kParts];
    auto load_b = [&](Frag(&b)[FN][kParts], int t) {
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int p = 0; p < kParts; ++p) b[j][p] = *(const Frag*)(Bl + ((size_t)(j * NSS + t) * kParts + p) * 512);
    };
    load_b(bq[0], 0);
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        if (t + 1 < NS) load_b(bq[(t + 1) & 1], t + 1);
        asm volatile("" ::: "memory");           // the loads stay ahead of the products
        const char* tile = As + t * (kParts * BM * 64);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            Frag af[kParts];
#pragma unroll
            for (int p = 0; p < kParts; ++p)
                af[p] = *(const Frag*)(tile + split_at(BM, p, i * 16 + (lane & 15), lane >> 4));
            split_mma(acc[i], bq[t & 1], af);
        }
    }
}

// four values of row r at columns c .. c + 3 (c % 4 == 0) of the step tiles
template <int BM> __device__ inline char* split_quad(char* T, int p, int r, int c) {
    return T + (c >> 5) * (kParts * BM * 64) + split_at(BM, p, r, (c >> 3) & 3) + (c & 4) * 2;
}
template <int BM> __device__ inline void put_quad(char* T, int r, int c, const float v[4]) {
    uint2 o[kParts];
    split2(v[0], v[1], o[0].x, o[1].x, o[2].x);
    split2(v[2], v[3], o[0].y, o[1].y, o[2].y);
#pragma unroll
    for (int p = 0; p < kParts; ++p) *(uint2*)split_quad<BM>(T, p, r, c) = o[p];
}
template <int BM> __device__ inline void get_quad(char* T, int r, int c, float v[4]) {
    uint2 o[kParts];
#pragma unroll
    for (int p = 0; p < kParts; ++p) o[p] = *(const uint2*)split_quad<BM>(T, p, r, c);
    auto sum = [](uint32_t h, uint32_t m, uint32_t l) {
        return __uint_as_float(h) + (__uint_as_float(m) + __uint_as_float(l));
    };
    v[0] = sum(o[0].x << 16, o[1].x << 16, o[2].x << 16);
    v[1] = sum(o[0].x & 0xffff0000u, o[1].x & 0xffff0000u, o[2].x & 0xffff0000u);
    v[2] = sum(o[0].y << 16, o[1].y << 16, o[2].y << 16);
    v[3] = sum(o[0].y & 0xffff0000u, o[1].y & 0xffff0000u, o[2].y & 0xffff0000u);
}

template <int BM, int H1, int H2, int H3>
__global__ __launch_bounds__(256, 2) void k_tailx(SplitTailArgs g) {
    typedef SplitTail<H1, H2, H3, BM> Sh;
    constexpr int NT = 256, FM = BM / 16;
    extern __shared__ __align__(16) char smem[];
    char *Hs = smem, *Us = smem + Sh::h2;                 // H2 / DZ2; DZ3 (H1 over both)
    float* sb2 = (float*)(smem + Sh::acts);               // b2 [H2], b3 [H3], w4 [H3]
    float *sb3 = sb2 + H2, *sw4 = sb3 + H3, *red = sw4 + H3;   // red [BM][4]

    // XCD-contiguous ranges over (model, row tile), as in k_tail
    const int nm = g.info->rows / BM, lin = xcd_tile(nm * g.M);
    if (lin < 0) return;
    const int z = lin / nm, row0 = lin % nm * BM;
    const int s = g.tile_species[row0 / g.row_tile];
    if (s < 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave;
    const size_t sz = (size_t)s * g.M + z;
    const float* Hrow = g.H1 + (size_t)row0 * g.ldh + (size_t)z * H1;

    for (int t = tid; t < BM * (H1 / 8); t += NT) {
        const int r = t / (H1 / 8), c = t % (H1 / 8);
        float v[8];
        *(float4*)&v[0] = *(const float4*)(Hrow + (size_t)r * g.ldh + c * 8);
        *(float4*)&v[4] = *(const float4*)(Hrow + (size_t)r * g.ldh + c * 8 + 4);
        uint4 o[kParts];
        split8(v, o);
#pragma unroll
        for (int p = 0; p < kParts; ++p) *(uint4*)(smem + (c >> 2) * Sh::tile + split_at(BM, p, r, c & 3)) = o[p];
    }
    for (int t = tid; t < H2 + 2 * H3; t += NT)
        sb2[t] = t < H2 ? g.b2[sz * H2 + t] : (t < H2 + H3 ? g.b3[sz * g.H3s + (t - H2)] : g.w4[sz * g.H3s + (t - H2 - H3)]);
    __syncthreads();
    const int rl = lane & 15, cl = 4 * (lane >> 4);

    // ---- layer 2 forward
    {
        constexpr int FN = H2 / 64;
        f32x4 acc[FM][FN];
        const int n0 = wn * (H2 / 4);
        split_product<BM, FM, FN, H1, H1>(acc, smem, g.W2x + sz * (kParts * H2 * H1), n0 / 16, lane, sb2 + n0 + cl);
        __syncthreads();   // every wave is done with the H1 tile, which H2 overwrites
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                float v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = celu(acc[i][j][q], g.alpha, g.inv_alpha);
                put_quad<BM>(Hs, rl + i * 16, n0 + j * 16 + cl, v);
            }
    }
    __syncthreads();   // H2 complete
    // ---- layer 3 forward, output layer, dE/dz3: the column tiles dealt to
    // the quarters as evenly as they go (160: 2, 3, 2, 3)
    {
        constexpr int F3 = H3 / 16, FNX = (F3 + 3) / 4;
        const int f0 = (wn * F3) / 4, fn = ((wn + 1) * F3) / 4 - f0;
        auto layer3 = [&](auto fn_c) {
            constexpr int FN = decltype(fn_c)::value;
            f32x4 acc[FM][FN];
            const int n0 = 16 * f0;
            split_product<BM, FM, FN, H2, H2>(acc, Hs, g.W3x + sz * (kParts * H2) * g.H3s, f0, lane, sb3 + n0 + cl);
            float part[FM] = {};
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int c = n0 + j * 16 + cl;
                float ww[4], wg[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    ww[q] = sw4[c + q];
                    wg[q] = ww[q] * g.gscale;
                }
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        part[i] += ww[q] * celu(acc[i][j][q], g.alpha, g.inv_alpha);
                        v[q] = dcelu_z(acc[i][j][q], g.inv_alpha) * wg[q];
                    }
                    put_quad<BM>(Us, rl + i * 16, c, v);
                }
            }
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                float v = part[i];
                v += __shfl_xor(v, 16);
                v += __shfl_xor(v, 32);
                if (lane < 16) red[(rl + i * 16) * 4 + wn] = v;
            }
        };
        if (fn == FNX || F3 % 4 == 0) layer3(std::integral_constant<int, FNX>{});
        else layer3(std::integral_constant<int, (FNX > 1 ? FNX - 1 : 1)>{});
    }
    __syncthreads();   // DZ3 and the energy partials complete
    if (tid < BM)
        g.epart[(size_t)(row0 + tid) * g.M + z] = red[tid * 4] + red[tid * 4 + 1] + red[tid * 4 + 2] + red[tid * 4 + 3];
    // ---- layer 3 backward: DZ2 = (DZ3 W3) celu'(H2), in place of H2 (each
    // lane reads and then overwrites only its own elements)
    {
        constexpr int FN = H2 / 64;
        f32x4 acc[FM][FN];
        const int n0 = wn * (H2 / 4);
        // the stored reduction length is the padded width of layer 3
        const bf16_t* W = g.W3Tx + sz * (kParts * H2) * g.H3s;
        split_product<BM, FM, FN, H3, (H3 + 63) / 64 * 64>(acc, Us, W, n0 / 16, lane, nullptr);
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                float hh[4], v[4];
                get_quad<BM>(Hs, rl + i * 16, n0 + j * 16 + cl, hh);
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = acc[i][j][q] * dcelu_h(hh[q], g.inv_alpha);
                put_quad<BM>(Hs, rl + i * 16, n0 + j * 16 + cl, v);
            }
    }
    __syncthreads();   // DZ2 complete
    // ---- layer 2 backward: DZ1 = (DZ2 W2) celu'(H1) -> HBM, H1 read again
    // (from L2) during the product
    {
        constexpr int FN = H1 / 64;
        f32x4 acc[FM][FN];
        const int n0 = wn * (H1 / 4);
        float hh[FM][FN][4];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                Quad<float, 1>::ld(Hrow + (size_t)(rl + i * 16) * g.ldh + n0 + j * 16 + cl, hh[i][j]);
        split_product<BM, FM, FN, H2, H2>(acc, Hs, g.W2Tx + sz * (kParts * H1 * H2), n0 / 16, lane, nullptr);
        float* Out = g.DZ1 + (size_t)row0 * g.ldh + (size_t)z * H1;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                float v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = acc[i][j][q] * dcelu_h(hh[i][j][q], g.inv_alpha);
                Quad<float, 1>::st(Out + (size_t)(rl + i * 16) * g.ldh + n0 + j * 16 + cl, v);
            }
    }
}

template <int BM, int H3>
static hipError_t run_tailx(const Shape& sh, const SplitTailArgs& a0, hipStream_t st, const Timer& tm) {
    constexpr int H1 = kTailH1, H2 = kTailH2;
    constexpr size_t lds = SplitTail<H1, H2, H3, BM>::lds_bytes;
    static_assert(lds <= 160 * 1024, "LDS of the split tail");
    SplitTailArgs a = a0;
    if (sh.Rcap % BM || sh.row_tile % BM) return hipErrorInvalidValue;
    auto kern = k_tailx<BM, H1, H2, H3>;
    hipError_t e = ensure_lds((const void*)kern, lds);
    if (e != hipSuccess) return e;
    tm.b("mlp_tail", st);
    hipLaunchKernelGGL(kern, dim3(sh.Rcap / BM * sh.M), dim3(256), lds, st, a);
    tm.e("mlp_tail", st);
    return hipGetLastError();
}

hipError_t split_tail(const Shape& sh, const DevWeights<PrecF32>& wt, Work<PrecF32>& w, hipStream_t st, const Timer& tm) {
    SplitTailArgs a{};
    a.H1 = w.H1; a.DZ1 = w.DZ1; a.ldh = sh.M * sh.H1;
    a.W2x = wt.W2x; a.W2Tx = wt.W2Tx; a.b2 = wt.b2;
    a.W3x = wt.W3x; a.W3Tx = wt.W3Tx; a.b3 = wt.b3; a.w4 = wt.w4;
    a.epart = w.Epart;
    a.gscale = (float)(sh.energy_scale / sh.M);
    a.alpha = (float)sh.celu_alpha;
    a.inv_alpha = (float)(1.0 / sh.celu_alpha);
    a.M = sh.M;
    a.H3s = sh.H3;
    a.tile_species = w.tile_species; a.row_tile = sh.row_tile;
    a.info = w.info;
    const bool n160 = sh.h3_used <= 160;   // layer 3 of at most 160 outputs (ANI-2x)
    return n160 ? run_tailx<32, 160>(sh, a, st, tm) : run_tailx<32, 192>(sh, a, st, tm);
}

template <int EPI>
hipError_t split_gemm(SplitArgs a, int R, int N, int nz, hipStream_t st, const Timer& tm, const char* name) {
    a.g.nz = nz;
    // 16-row buckets (at most 256 atoms): K split over four waves.  One 64-atom
    // ligand, 8 models: 16.6 / 15.1 us forward / backward (k_gemm on FP32 MFMAs
    // 17.1 / 18.4), 59 MB of weights each, near the rate a copy reaches; eight
    // waves or 16-column tiles 17-21 us.  (Layer 3's energy partials are
    // counted per 64 columns.)
    if (a.g.row_tile == 16) {
        if (EPI == EPI_L3F) return run_gxk<1, 4, 4, 1, EPI>(a, R, N, st, tm, name);
        if (a.g.K >= 2048) return run_gxk<1, 4, 4, 2, EPI>(a, R, N, st, tm, name);
        if (a.g.K >= 512) return run_gxk<1, 2, 4, 4, EPI>(a, R, N, st, tm, name);
        return run_gxk<1, 2, 4, 2, EPI>(a, R, N, st, tm, name);
    }
    const int tiles = R / 64 * nz;   // of this call: the column tiles below give the same sums bit for bit
    if (EPI == EPI_L3F) return run_gx<4, 1, 4, EPI>(a, R, N, st, tm, name);
    // long K and at most one workgroup per CU: K split over eight waves (the
    // layer-1 backward of 569 atoms 34 us, 40 on the tile below, 55 on 128
    // columns; at two rounds, 848 atoms, 58 against 51).  The split changes the
    // roundings, so the handle's capacity decides where results must not depend
    // on what else, or which bounds, a call has (pick_rows)
    if (a.g.K >= 1024 && a.g.pick_rows / 64 * nz * (N / 64) <= 256) return run_gxk<4, 4, 8, 2, EPI>(a, R, N, st, tm, name);
    // 128 columns where they give about three workgroups per two CUs (3,445
    // atoms, forward / backward: 93 / 97 us, 256 columns 93 / 106; 12,011:
    // 235 / 267 against 252 / 292; 47,999: 817 / 891 against 880 / 900), 64
    // where they don't (848 atoms: 38 / 51 us against 46 / 57; 2,403 atoms'
    // backward 80 against 91)
    if (N % 128 == 0 && tiles * (N / 128) >= 384) return run_gx<4, 2, 4, EPI>(a, R, N, st, tm, name);
    if (N % 192 == 0 && tiles * (N / 192) >= 256) return run_gx<4, 3, 4, EPI>(a, R, N, st, tm, name);
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
