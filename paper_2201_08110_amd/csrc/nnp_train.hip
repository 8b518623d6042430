// nnp_train.hip -- parameter gradients of a loss L(E, F) for training.
//
// F = -dE/dx (Methods, Eq. 3), so for cotangents gE = dL/dE and gF = dL/dF
//   dL/dW = sum_b gE_b dE_b/dW - d/dW sum_i (dE/dG_i . Gdot_i),
// with Gdot = (dG/dx) gF the AEV tangent (independent of the weights).  Per
// atom and model the inner product is (u/M) times the tangent of the network
// output along Gdot_i, so every network is differentiated through its primal
// and tangent graph with output adjoints alpha = (u/M) gE_b (primal) and
// beta = -u/M (tangent).  This file holds the elementwise layer-3 reverse
// step, the weight-gradient reductions over each element bucket's rows and
// the bias / output-layer sums; the GEMM steps live in nnp_mlp.hip.
#include "nnp_split.h"

namespace nnp {

template <typename TA> __device__ inline TA dcelu_h_(TA h, TA al) { return h >= TA(0) ? TA(1) : TA(1) + h / al; }

// per-row output adjoints (zero on padding rows)
template <typename TA>
__device__ inline void row_adjoints(int r, const int32_t* __restrict__ atom_of_row,
                                    const int32_t* __restrict__ mol_of_atom,
                                    const double* __restrict__ grad_E, bool has_gF, double scale,
                                    TA& al, TA& be) {
    const int a = atom_of_row[r];
    al = TA(0);
    be = TA(0);
    if (a >= 0) {
        if (grad_E) al = (TA)(scale * grad_E[mol_of_atom[a]]);
        if (has_gF) be = (TA)(-scale);
    }
}

// layer-3 adjoints: zbar3 = w4 (alpha CELU'(z3) + beta (CELU''/CELU')(z3) hdot3),
// zdotbar3 = w4 beta CELU'(z3)
template <typename P>
__global__ __launch_bounds__(256) void k_rev3(int M, int H3, double scale, double celu_alpha,
                                              bool has_gF, const BucketInfo* __restrict__ info,
                                              const int32_t* __restrict__ tile_species, int row_tile,
                                              const int32_t* __restrict__ atom_of_row,
                                              const int32_t* __restrict__ mol_of_atom,
                                              const double* __restrict__ grad_E,
                                              const typename P::TA* __restrict__ w4,
                                              const typename P::TS* __restrict__ Hh,
                                              const typename P::TS* __restrict__ Th,
                                              typename P::TS* __restrict__ ZB,
                                              typename P::TS* __restrict__ ZDB) {
    typedef typename P::TA TA;
    typedef typename P::TS TS;
    const int r = blockIdx.x;
    if (r >= info->rows) return;
    const int s = tile_species[r / row_tile];
    if (s < 0) return;
    TA al, be;
    row_adjoints(r, atom_of_row, mol_of_atom, grad_E, has_gF, scale / M, al, be);
    const TA ca = (TA)celu_alpha;
    const size_t base = (size_t)r * M * H3;
    for (int e = threadIdx.x; e < M * H3; e += blockDim.x) {
        const int m = e / H3, n = e % H3;
        const TA w = w4[((size_t)s * M + m) * H3 + n];
        const TA h = Store<TS>::ld(Hh[base + e]);
        const TA hd = has_gF ? Store<TS>::ld(Th[base + e]) : TA(0);
        const TA d1 = dcelu_h_(h, ca);
        const TA rho = h < TA(0) ? TA(1) / ca : TA(0);
        ZB[base + e] = Store<TS>::st(w * (al * d1 + be * rho * hd));
        ZDB[base + e] = Store<TS>::st(w * be * d1);
    }
}

template <typename P>
hipError_t launch_train_rev3(const Shape& sh, const DevWeights<P>& wt, Work<P>& w,
                             TrainWork<P>& tw, const int32_t* mol_of_atom, const double* grad_E,
                             bool has_gF, hipStream_t st, const Timer& tm) {
    tm.b("train_rev3", st);
    hipLaunchKernelGGL(k_rev3<P>, dim3(sh.Rcap), dim3(256), 0, st, sh.M, sh.H3, sh.energy_scale,
                       sh.celu_alpha, has_gF, w.info, w.tile_species, sh.row_tile, w.atom_of_row,
                       mol_of_atom, grad_E, wt.w4, tw.H3, tw.TH3, w.DZ3, tw.ZDB3);
    tm.e("train_rev3", st);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Weight gradient of one layer for every (element, model):
//   Wbar[n][k] = sum over the element's bucket rows r of
//                X1[r][xo + n] Y1[r][yo + k] + X2[r][xo + n] Y2[r][yo + k]
// (xo = m * out width, yo = m * in width or 0 for the AEV operands),
// written into the packed gradient array.  FP64: MFMA 16x16x4 takes one
// element per lane, so the row-major tiles feed it without a transpose: the
// reduction runs over rows, 16 per LDS slice.  (FP32: k_wgx.)
struct MFW {
    typedef f64x4 Acc;
    __device__ static Acc mma(double a, double b, Acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row(int l, int r) { return (l >> 4) + 4 * r; }
};

constexpr int kWT = 64;   // output tile (n and k)
constexpr int kWR = 16;   // rows per LDS slice (divides every row tile)

// One workgroup: a 64 x 64 tile of one (element, model) weight gradient,
// 2 x 2 waves of 32 x 32 (many workgroups: the reduction over a bucket's rows
// is serial in each).  The next 16-row slice of both operands is loaded into
// registers (16-byte vectors) while the MFMAs consume the current one from
// LDS.  Columns past an operand's valid width read as zero.
template <typename P>
__global__ __launch_bounds__(256) void k_wgrad(int S, int M, const BucketInfo* __restrict__ info,
                                               const typename P::TS* __restrict__ X1,
                                               const typename P::TS* __restrict__ Y1,
                                               const typename P::TS* __restrict__ X2,
                                               const typename P::TS* __restrict__ Y2, int ldx,
                                               int ldy, int xw, int yw, int out_o, int in_o,
                                               long offW, long net, int ntn,
                                               typename P::TA* __restrict__ gparam) {
    typedef typename P::TS TS;
    typedef typename P::TA TA;
    typedef MFW mf;
    constexpr int VEC = 16 / (int)sizeof(TS);            // elements per 16-byte load
    constexpr int LD = kWT + VEC;                        // padded LDS row
    constexpr int NV = kWR * kWT / VEC / 256;            // vector loads per thread and operand
    constexpr int FM = kWT / 32, FN = kWT / 32;          // 16 x 16 MFMA tiles per wave
    typedef double2 TV;
    __shared__ __align__(16) TS Xs[kWR][LD];
    __shared__ __align__(16) TS Ys[kWR][LD];
    const int tile = blockIdx.x, sm = blockIdx.y;
    const int s = sm % S, m = sm / S;
    const int tn = tile % ntn, tk = tile / ntn;
    const int n0 = tn * kWT, k0 = tk * kWT;
    if (n0 >= out_o || k0 >= in_o) return;
    const int r0 = info->off[s], r1 = info->off[s + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int xv = xw, yv = yw ? yw : ldy;               // valid columns of each operand block
    typename mf::Acc acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = 0;
    const int xo = m * xw + n0, yo = m * yw + k0;
    TV xr[NV], yr[NV];
    auto gload = [&](const TS* X, const TS* Y, int r) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int e = tid + 256 * v, rr = e / (kWT / VEC), col = (e % (kWT / VEC)) * VEC;
            TV zx, zy;
            zx = zy = TV{};
            xr[v] = n0 + col < xv ? *(const TV*)(X + (size_t)(r + rr) * ldx + xo + col) : zx;
            yr[v] = k0 + col < yv ? *(const TV*)(Y + (size_t)(r + rr) * ldy + yo + col) : zy;
        }
    };
    auto lstore = [&]() {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int e = tid + 256 * v, rr = e / (kWT / VEC), col = (e % (kWT / VEC)) * VEC;
            *(TV*)&Xs[rr][col] = xr[v];
            *(TV*)&Ys[rr][col] = yr[v];
        }
    };
    for (int pass = 0; pass < 2; ++pass) {
        const TS* X = pass ? X2 : X1;
        const TS* Y = pass ? Y2 : Y1;
        if (!X || !Y || r0 >= r1) continue;
        gload(X, Y, r0);
        for (int r = r0; r < r1; r += kWR) {
            lstore();
            __syncthreads();
            if (r + kWR < r1) gload(X, Y, r + kWR);
#pragma unroll
            for (int kk = 0; kk < kWR; kk += 4) {
                const int kr = kk + (lane >> 4);
                TS a[FM], b[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) a[i] = Xs[kr][wm * (kWT / 2) + i * 16 + (lane & 15)];
#pragma unroll
                for (int j = 0; j < FN; ++j) b[j] = Ys[kr][wn * (kWT / 2) + j * 16 + (lane & 15)];
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) acc[i][j] = mf::mma(a[i], b[j], acc[i][j]);
            }
            __syncthreads();
        }
    }
    TA* out = gparam + ((long)m * S + s) * net + offW;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + wm * (kWT / 2) + i * 16 + mf::row(lane, q);
                const int k = k0 + wn * (kWT / 2) + j * 16 + (lane & 15);
                if (n < out_o && k < in_o) out[(long)n * in_o + k] = (TA)acc[i][j][q];
            }
}

// Column sums over each element bucket: the bias gradients (adjoints of layers
// 1-3), the output layer's weights (rows weighted by their output adjoints)
// and its bias.  One launch: a workgroup takes 32 columns of one (element,
// model) with 32 row groups, so a bucket of 1,600 rows is 50 strided loads a
// thread, eight in flight, and a fixed tree over the groups; the row weights,
// each a chain of three dependent loads, are fetched 1,024 rows at a time
// into LDS.  64 columns x 4 row groups in four launches were bound by that
// chain: 855 us a training step of 3,520 atoms, now 38 us.
constexpr int kSumCols = 32, kSumGroups = 32, kSumRows = kSumCols * kSumGroups;
template <typename P> struct SumArgs {
    const typename P::TS* X[3];   // adjoints of layers 1-3
    int ld[3], xw[3], out[3], nb[3];
    long off[3];
    const typename P::TS *Hh, *Th;   // layer-3 activations and tangents
    int H3, o3;
    double scale;
    bool has_gF;
    const int32_t *atom_of_row, *mol_of_atom;
    const double* grad_E;
    long offw4, offb4, net;
};

template <typename P>
__global__ __launch_bounds__(kSumRows) void k_row_sums(int S, int M, const BucketInfo* __restrict__ info, SumArgs<P> g,
                                                       typename P::TA* __restrict__ gparam) {
    typedef typename P::TA TA;
    typedef typename P::TS TS;
    __shared__ TA part[kSumGroups][kSumCols + 1];
    __shared__ TA wal[kSumRows], wbe[kSumRows];
    const int s = blockIdx.y / M, m = blockIdx.y % M;
    int blk = blockIdx.x, layer = 0;
    while (layer < 3 && blk >= g.nb[layer]) blk -= g.nb[layer++];
    const int c = threadIdx.x % kSumCols, rg = threadIdx.x / kSumCols, col = blk * kSumCols + c;
    const int r0 = info->off[s], r1 = info->off[s + 1];
    TA* out = gparam + ((long)m * S + s) * g.net;
    TA acc = 0, accb = 0;
    if (layer < 3) {
        if (col < g.out[layer]) {
            const TS* X = g.X[layer] + (size_t)m * g.xw[layer] + col;
            const size_t ld = g.ld[layer];
#pragma unroll 8
            for (int r = r0 + rg; r < r1; r += kSumGroups) acc += Store<TS>::ld(X[r * ld]);
        }
    } else {
        const size_t ld = (size_t)M * g.H3, at = (size_t)m * g.H3 + min(col, g.H3 - 1);
        for (int rc = r0; rc < r1; rc += kSumRows) {
            __syncthreads();
            const int r = rc + (int)threadIdx.x;
            TA al = 0, be = 0;
            if (r < r1) row_adjoints(r, g.atom_of_row, g.mol_of_atom, g.grad_E, g.has_gF, g.scale / M, al, be);
            wal[threadIdx.x] = al;
            wbe[threadIdx.x] = be;
            accb += al;
            __syncthreads();
            const int n = min(kSumRows, r1 - rc);
#pragma unroll 4
            for (int t = rg; t < n; t += kSumGroups) {
                const size_t e = (size_t)(rc + t) * ld + at;
                acc += wal[t] * Store<TS>::ld(g.Hh[e]) + (g.has_gF ? wbe[t] * Store<TS>::ld(g.Th[e]) : TA(0));
            }
        }
    }
    auto tree = [&](TA v) {   // column sums over the row groups, left in part[0]
        part[rg][c] = v;
        for (int o = kSumGroups / 2; o > 0; o >>= 1) {
            __syncthreads();
            if (rg < o) part[rg][c] += part[rg + o][c];
        }
        __syncthreads();
    };
    tree(acc);
    const int o_w = layer < 3 ? g.out[layer] : g.o3;
    const long o_at = layer < 3 ? g.off[layer] : g.offw4;
    if (rg == 0 && col < o_w) out[o_at + col] = part[0][c];
    if (layer == 3 && blk == 0) {   // each thread's rows' weights: the sum over every row
        __syncthreads();
        tree(accb);
        if (threadIdx.x == 0) {
            TA v = 0;
            for (int q = 0; q < kSumCols; ++q) v += part[0][q];
            out[g.offb4] = v;
        }
    }
}

// The same weight gradients in FP32 on the bf16 matrix cores, both operands
// split into three bf16 parts (nnp_split.h) on their way into LDS, transposed:
// the reduction runs over rows, 32 a step, so a thread takes 8 rows x 2
// columns of each operand and writes one 16-byte chunk (8 rows) a column and
// part.  A workgroup owns a 128 x 128 tile (2 x 2 waves of 64 x 64) of one
// (element, model, layer); all three layers' tiles are one launch, the
// elements in index order (the commonest first), so the short chains of the
// rare ones fill in behind the long ones.  Bound by LDS reads (24 KiB per
// wave and step for 96 MFMAs).  Training step of 3,520 atoms: three FP32 MFMA
// launches of 64 x 64 tiles 701 us, this one 242 us.
struct WgLayer {
    const float *X1, *Y1, *X2, *Y2;   // Wbar = X1^T Y1 + X2^T Y2 over the bucket's rows
    int ldx, ldy, xw, yw;             // leading dimensions; columns per model (yw 0: shared by all)
    int out_o, in_o, ntn, nt;         // gradient [out_o][in_o]; tiles along n and per model
    long offW;
};
struct WgArgs {
    WgLayer l[3];
};
constexpr int kXT = 128;

__global__ __launch_bounds__(256, 2) void k_wgx(int S, int M, const BucketInfo* __restrict__ info, WgArgs w, long net,
                                                float* __restrict__ gparam) {
    typedef bf16x8 Frag;
    __shared__ __align__(16) char lds[2][kParts * kXT * 64];
    int blk = blockIdx.x, li = 0;
    while (blk >= w.l[li].nt * M) blk -= w.l[li++].nt * M;
    const WgLayer& g = w.l[li];
    const int s = blockIdx.y, m = blk / g.nt, tile = blk % g.nt;
    const int n0 = (tile % g.ntn) * kXT, k0 = (tile / g.ntn) * kXT;
    const int r0 = info->off[s], r1 = info->off[s + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int cp = 2 * lane;                              // this thread's two columns, rows 8 wave ..
    // columns past an operand's width repeat its last two (their products are
    // not stored)
    const int xc = min(n0 + cp, g.xw - 2), yc = min(k0 + cp, (g.yw ? g.yw : g.ldy) - 2);
    const size_t xo = (size_t)m * g.xw + xc, yo = (size_t)m * g.yw + yc;
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;
    float2 xr[8], yr[8];
    auto load = [&](const float* X, const float* Y, int r) {
        // buckets are whole multiples of 16 rows: past the end the last eight
        // again, against zeros
        const bool in = r + 8 * wave < r1;
        const size_t row = min(r + 8 * wave, r1 - 8);
        const float *xp = X + row * g.ldx + xo, *yp = Y + row * g.ldy + yo;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            xr[q] = *(const float2*)(xp + (size_t)q * g.ldx);
            yr[q] = *(const float2*)(yp + (size_t)q * g.ldy);
        }
        if (!in)
#pragma unroll
            for (int q = 0; q < 8; ++q) xr[q] = make_float2(0.f, 0.f);
    };
    auto store = [&](char* t, const float2(&v)[8]) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float e[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) e[q] = c ? v[q].y : v[q].x;
            uint4 o[kParts];
            split8(e, o);
#pragma unroll
            for (int p = 0; p < kParts; ++p) *(uint4*)(t + split_at(kXT, p, cp + c, wave)) = o[p];
        }
    };
    for (int pass = 0; pass < 2; ++pass) {
        const float* X = pass ? g.X2 : g.X1;
        const float* Y = pass ? g.Y2 : g.Y1;
        if (!X || !Y || r0 >= r1) continue;
        load(X, Y, r0);
        for (int r = r0; r < r1; r += 32) {
            store(lds[0], xr);
            store(lds[1], yr);
            __syncthreads();
            if (r + 32 < r1) load(X, Y, r + 32);
            asm volatile("" ::: "memory");                // keep those loads ahead of the products
            Frag bf[4][kParts];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int p = 0; p < kParts; ++p)
                    bf[j][p] = *(const Frag*)(lds[1] + split_at(kXT, p, wn * 64 + j * 16 + (lane & 15), lane >> 4));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                Frag af[kParts];
#pragma unroll
                for (int p = 0; p < kParts; ++p)
                    af[p] = *(const Frag*)(lds[0] + split_at(kXT, p, wm * 64 + i * 16 + (lane & 15), lane >> 4));
                split_mma(acc[i], bf, af);
            }
            __syncthreads();
        }
    }
    float* out = gparam + ((long)m * S + s) * net + g.offW;
    auto write = [&](auto whole) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = n0 + wm * 64 + i * 16 + (lane & 15), k = k0 + wn * 64 + j * 16 + 4 * (lane >> 4) + q;
                    if (whole.value || (n < g.out_o && k < g.in_o)) out[(long)n * g.in_o + k] = acc[i][j][q];
                }
    };
    if (n0 + kXT <= g.out_o && k0 + kXT <= g.in_o) write(std::true_type{});
    else write(std::false_type{});
}

template <typename P>
hipError_t launch_train_grads(const Shape& sh, const NetLayout& nl, Work<P>& w, TrainWork<P>& tw,
                              const int32_t* mol_of_atom, const double* grad_E, bool has_gF,
                              typename P::TA* gp, hipStream_t st, const Timer& tm) {
    typedef typename P::TS TS;
    const int S = sh.S, M = sh.M, H1 = sh.H1, H2 = sh.H2, H3 = sh.H3, Dp = sh.Dp;
    const dim3 blk(256);
    tm.b("train_wgrad", st);
    // W1 [o1 x D] from (ZB1, G) + (ZDB1, GD), W2 [o2 x o1] from (ZB2, H1) +
    // (ZDB2, TH1), W3 [o3 x o2] from (ZB3, H2) + (ZDB3, TH2)
    if constexpr (std::is_same<P, PrecF32>::value) {
        WgArgs a{};
        auto layer = [&](int i, const float* X1, const float* Y1, const float* X2, const float* Y2, int xw, int yw,
                         int ldy, int out_o, int in_o, long offW) {
            const int ntn = (out_o + kXT - 1) / kXT;
            a.l[i] = {X1, Y1, has_gF ? X2 : nullptr, Y2, M * xw, ldy, xw, yw, out_o, in_o, ntn,
                      ntn * ((in_o + kXT - 1) / kXT), offW};
        };
        layer(0, w.DZ1, w.G, tw.ZDB1, tw.GD, H1, 0, Dp, nl.o1, nl.D, nl.offW1);
        layer(1, w.DZ2, w.H1, tw.ZDB2, tw.TH1, H2, H1, M * H1, nl.o2, nl.o1, nl.offW2);
        layer(2, w.DZ3, w.H2, tw.ZDB3, tw.TH2, H3, H2, M * H2, nl.o3, nl.o2, nl.offW3);
        hipLaunchKernelGGL(k_wgx, dim3((a.l[0].nt + a.l[1].nt + a.l[2].nt) * M, S), blk, 0, st, S, M, w.info, a, nl.net, gp);
    } else {
        auto layer = [&](const TS* X1, const TS* Y1, const TS* X2, const TS* Y2, int xw, int yw, int ldy, int out_o,
                         int in_o, long offW) {
            const int ntn = (out_o + kWT - 1) / kWT, ntk = (in_o + kWT - 1) / kWT;
            hipLaunchKernelGGL(k_wgrad<P>, dim3(ntn * ntk, S * M), blk, 0, st, S, M, w.info, X1, Y1,
                               has_gF ? X2 : nullptr, Y2, M * xw, ldy, xw, yw, out_o, in_o, offW, nl.net, ntn, gp);
        };
        layer(w.DZ3, w.H2, tw.ZDB3, tw.TH2, H3, H2, M * H2, nl.o3, nl.o2, nl.offW3);
        layer(w.DZ2, w.H1, tw.ZDB2, tw.TH1, H2, H1, M * H1, nl.o2, nl.o1, nl.offW2);
        layer(w.DZ1, w.G, tw.ZDB1, tw.GD, H1, 0, Dp, nl.o1, nl.D, nl.offW1);
    }
    // biases and the output layer
    SumArgs<P> a{};
    const TS* X[3] = {w.DZ1, w.DZ2, w.DZ3};
    const int xw[3] = {H1, H2, H3}, out[3] = {nl.o1, nl.o2, nl.o3};
    const long off[3] = {nl.offb1, nl.offb2, nl.offb3};
    int nb = (nl.o3 + kSumCols - 1) / kSumCols;
    for (int i = 0; i < 3; ++i) {
        a.X[i] = X[i];
        a.ld[i] = M * xw[i];
        a.xw[i] = xw[i];
        a.out[i] = out[i];
        a.nb[i] = (out[i] + kSumCols - 1) / kSumCols;
        a.off[i] = off[i];
        nb += a.nb[i];
    }
    a.Hh = tw.H3;
    a.Th = tw.TH3;
    a.H3 = H3;
    a.o3 = nl.o3;
    a.scale = sh.energy_scale;
    a.has_gF = has_gF;
    a.atom_of_row = w.atom_of_row;
    a.mol_of_atom = mol_of_atom;
    a.grad_E = grad_E;
    a.offw4 = nl.offw4;
    a.offb4 = nl.offb4;
    a.net = nl.net;
    hipLaunchKernelGGL(k_row_sums<P>, dim3(nb, S * M), dim3(kSumRows), 0, st, S, M, w.info, a, gp);
    tm.e("train_wgrad", st);
    return hipGetLastError();
}

template <typename TS>
__global__ void k_fill(TS* __restrict__ p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = TS(0);
}

template <typename P>
hipError_t launch_fill(typename P::TS* p, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill<typename P::TS>, dim3((unsigned)blocks), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

// dL/dx of an energy-only loss: sum_b gE_b dE_b/dx_i = -gE_b(i) F_i.  The
// molecule comes from the offsets (their last b with mol_off[b] <= i, always
// one of the B): an evaluation leaves no molecule for the atoms it refuses (a
// molecule above the capacity, offsets that do not end at the atom count).
template <typename T>
__global__ void k_grad_coords(int A, int B, const int32_t* __restrict__ mol_off,
                              const double* __restrict__ grad_E, const T* __restrict__ F,
                              T* __restrict__ gx) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 3 * A) return;
    double g = 0.0;
    if (grad_E) {
        int lo = 0, hi = B;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (mol_off[mid] <= i / 3) lo = mid;
            else hi = mid;
        }
        g = grad_E[lo];
    }
    gx[i] = (T)(-g * (double)F[i]);
}

template <typename P>
hipError_t launch_grad_coords(int A, int B, const int32_t* mol_off, const double* grad_E,
                              const typename P::T* F, typename P::T* gx, hipStream_t st) {
    if (A == 0) return hipSuccess;
    hipLaunchKernelGGL(k_grad_coords<typename P::T>, dim3((3 * A + 255) / 256), dim3(256), 0, st, A, B,
                       mol_off, grad_E, F, gx);
    return hipGetLastError();
}

// parameter gradients of element networks narrower than the padded layout:
// dst[i] = src[map[i]] (the padded entries are dropped)
template <typename TA>
__global__ void k_gather(int64_t n, const int32_t* __restrict__ map, const TA* __restrict__ src,
                         TA* __restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[map[i]];
}

template <typename TA>
hipError_t launch_gather(int64_t n, const int32_t* map, const TA* src, TA* dst, hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather<TA>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, map, src, dst);
    return hipGetLastError();
}
template hipError_t launch_gather<float>(int64_t, const int32_t*, const float*, float*, hipStream_t);
template hipError_t launch_gather<double>(int64_t, const int32_t*, const double*, double*, hipStream_t);

#define NNP_TRAIN_INST(P)                                                                       \
    template hipError_t launch_train_rev3<P>(const Shape&, const DevWeights<P>&, Work<P>&,     \
                                             TrainWork<P>&, const int32_t*, const double*,     \
                                             bool, hipStream_t, const Timer&);                 \
    template hipError_t launch_train_grads<P>(const Shape&, const NetLayout&, Work<P>&,         \
                                              TrainWork<P>&, const int32_t*, const double*,    \
                                              bool, P::TA*, hipStream_t, const Timer&);        \
    template hipError_t launch_fill<P>(P::TS*, size_t, hipStream_t);                           \
    template hipError_t launch_grad_coords<P>(int, int, const int32_t*, const double*, const P::T*, \
                                              P::T*, hipStream_t);
NNP_TRAIN_INST(PrecF64)
NNP_TRAIN_INST(PrecF32)
template hipError_t launch_fill<PrecBF16>(bf16_t*, size_t, hipStream_t);
template hipError_t launch_grad_coords<PrecBF16>(int, int, const int32_t*, const double*, const float*,
                                                 float*, hipStream_t);

}  // namespace nnp
