// nnp_params.hip -- device-side replacement of the network parameters.
//
// A training loop keeps its packed master parameters on the GPU (Methods,
// first optimisation: no CPU<->GPU copies per step); this kernel scatters
// them into every device layout the evaluation kernels read (the row-major
// and transposed matrices, the fragment-ordered copies, biases and output
// layer); nnp_create and nnp_set_weights upload host weights through it too,
// so a handle updated here computes bitwise what a handle created with the
// same weights does.
#include "nnp_split.h"

namespace nnp {

// FP32 matrix entries: infinite ones as the largest finite value, for their
// parts would be NaN against any feature (and zero past CELU); -infinity times
// a positive feature still ends in CELU's -alpha
__device__ inline float finite_weight(float v) { return isinf(v) ? copysignf(3.40282347e38f, v) : v; }

// a parameter as three bf16 parts at p[0], p[512], p[1024] (nnp_split.h)
__device__ inline void put_parts(bf16_t* p, float v) {
    const bf16_t h = (bf16_t)(__float_as_uint(v) >> 16);
    const float r = v - bf2f(h);
    const bf16_t m = Store<bf16_t>::st(r);
    p[0] = h;
    p[512] = m;
    p[1024] = Store<bf16_t>::st(r - bf2f(m));
}

template <typename P, typename TSRC>
__global__ __launch_bounds__(256) void k_set_params(int64_t first, int64_t n, const TSRC* __restrict__ src,
                                                    const int32_t* __restrict__ map, ParamPack pk,
                                                    DevWeights<P> dw) {
    typedef typename P::TS TS;
    typedef typename P::TA TA;
    constexpr bool f32 = std::is_same<P, PrecF32>::value;   // parts, no row-major matrices
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double v = (double)src[i];   // parameter first + i
    const TA va = (TA)v;
    if constexpr (f32) v = finite_weight(va);   // (va: biases and the output layer as they are)
    const TS vs = Store<TS>::st((TA)v);
    // position in the uniform (padded) packed layout: [m][s]{W1 b1 W2 b2 W3 b3 w4 b4}
    const int64_t pi = map ? (int64_t)map[first + i] : first + i;
    const int64_t ms = pi / pk.net;
    const int64_t r = pi - ms * pk.net;
    const int m = (int)(ms / pk.S), s = (int)(ms % pk.S);
    const int M = pk.M, H1 = pk.H1, H2 = pk.H2, H3 = pk.H3, Dp = pk.Dp;
    const size_t sm = (size_t)s * M + m;
    if (r < pk.offb1) {                       // W1 [o1][D]
        const int nn = (int)(r / pk.D), k = (int)(r % pk.D);
        const int col = m * H1 + nn, N1 = M * H1;
        if (f32 && dw.W1x) {
            put_parts(dw.W1x + (size_t)s * N1 * Dp * 3 + split_index(col, k, Dp), (float)v);
            put_parts(dw.W1Tx + (size_t)s * N1 * Dp * 3 + split_index(k, col, N1), (float)v);
        }
        if (!f32) {
            dw.W1[((size_t)s * N1 + col) * Dp + k] = vs;
            dw.W1T[((size_t)s * Dp + k) * N1 + col] = vs;
        }
        if (sizeof(TS) < 8) {
            dw.W1f[(size_t)s * N1 * Dp + frag_index<TS>(col, k, Dp)] = vs;
            dw.W1Tf[(size_t)s * N1 * Dp + frag_index<TS>(k, col, N1)] = vs;
        }
    } else if (r < pk.offW2) {                // b1 [o1]
        dw.b1[(size_t)s * M * H1 + (size_t)m * H1 + (r - pk.offb1)] = va;
    } else if (r < pk.offb2) {                // W2 [o2][o1]
        const int64_t q = r - pk.offW2;
        const int nn = (int)(q / pk.o1), k = (int)(q % pk.o1);
        if (f32 && dw.W2x) {
            put_parts(dw.W2x + sm * H2 * H1 * 3 + split_index(nn, k, H1), (float)v);
            put_parts(dw.W2Tx + sm * H1 * H2 * 3 + split_index(k, nn, H2), (float)v);
        }
        if (!f32) {
            dw.W2[(sm * H2 + nn) * H1 + k] = vs;
            dw.W2T[(sm * H1 + k) * H2 + nn] = vs;
        }
        dw.W2f[sm * H2 * H1 + frag_index<TS>(nn, k, H1)] = vs;
        dw.W2Tf[sm * H1 * H2 + frag_index<TS>(k, nn, H2)] = vs;
    } else if (r < pk.offW3) {                // b2 [o2]
        dw.b2[sm * H2 + (r - pk.offb2)] = va;
    } else if (r < pk.offb3) {                // W3 [o3][o2]
        const int64_t q = r - pk.offW3;
        const int nn = (int)(q / pk.o2), k = (int)(q % pk.o2);
        if (f32 && dw.W3x) {
            put_parts(dw.W3x + sm * H3 * H2 * 3 + split_index(nn, k, H2), (float)v);
            put_parts(dw.W3Tx + sm * H2 * H3 * 3 + split_index(k, nn, H3), (float)v);
        }
        if (!f32) {
            dw.W3[(sm * H3 + nn) * H2 + k] = vs;
            dw.W3T[(sm * H2 + k) * H3 + nn] = vs;
        }
        dw.W3f[sm * H3 * H2 + frag_index<TS>(nn, k, H2)] = vs;
        dw.W3Tf[sm * H2 * H3 + frag_index<TS>(k, nn, H3)] = vs;
    } else if (r < pk.offw4) {                // b3 [o3]
        dw.b3[sm * H3 + (r - pk.offb3)] = va;
    } else if (r < pk.offb4) {                // w4 [o3]
        dw.w4[sm * H3 + (r - pk.offw4)] = va;
    } else {                                  // b4
        dw.b4[sm] = va;
    }
}

template <typename P, typename TSRC>
hipError_t launch_set_params(int64_t first, int64_t n, const TSRC* src, const int32_t* map, const ParamPack& pk,
                             const DevWeights<P>& dw, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_set_params<P, TSRC>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, first, n,
                       src, map, pk, dw);
    return hipGetLastError();
}

// The same for a whole parameter array on FP32 handles, whose matrices are kept
// in fragment order and, split into bf16 parts, in fragment order again, each
// also transposed.  A workgroup takes a 64 x 64 piece of one matrix through
// LDS, so it reads rows and writes every layout in 1 KiB runs; one parameter a
// thread writes 2- and 4-byte pieces 16 bytes apart.  Bound by the stores
// (8 or 20 bytes a parameter): 19 M parameters, 304 us that way, 90 this.
template <typename TSRC>
__global__ __launch_bounds__(256) void k_set_nets(const TSRC* __restrict__ src, ParamPack pk,
                                                  DevWeights<PrecF32> dw) {
    __shared__ float t[64][65];
    const int m = blockIdx.y / pk.S, s = blockIdx.y % pk.S;
    const size_t sm = (size_t)s * pk.M + m;
    int64_t base = 0;   // this network's place in the packed array
    for (int q = 0; q < pk.S; ++q) {
        const int* w = pk.w[q];
        const int64_t n = (int64_t)w[1] * (w[0] + 1) + (int64_t)w[2] * (w[1] + 1) + (int64_t)w[3] * (w[2] + 1) + w[3] + 1;
        base += (m + (q < s)) * n;
    }
    src += base;
    const int* w = pk.w[s];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // which matrix (l = 1..3), or the vectors (l = 4)
    const int np[4] = {pk.Dp, pk.H1, pk.H2, pk.H3};
    int blk = blockIdx.x, l = 1;
    int64_t off = 0;
    for (; l < 4; ++l) {
        const int nt = np[l] / 64 * (np[l - 1] / 64);
        if (blk < nt) break;
        blk -= nt;
        off += (int64_t)w[l] * (w[l - 1] + 1);
    }
    if (l == 4) {
        int64_t o = 0;
        for (int q = 1; q < 4; ++q) {
            o += (int64_t)w[q] * w[q - 1];
            float* b = (q == 1 ? dw.b1 : q == 2 ? dw.b2 : dw.b3) + sm * np[q];
            for (int i = tid; i < w[q]; i += 256) b[i] = (float)src[o + i];
            o += w[q];
        }
        for (int i = tid; i < w[3]; i += 256) dw.w4[sm * pk.H3 + i] = (float)src[o + i];
        if (tid == 0) dw.b4[sm] = (float)src[o + w[3]];
        return;
    }
    const int N = np[l], K = np[l - 1], nkb = K / 64, n0 = blk / nkb * 64, k0 = blk % nkb * 64;
    src += off;
    for (int r = wave; r < 64; r += 4)
        t[r][lane] = n0 + r < w[l] && k0 + lane < w[l - 1] ? finite_weight((float)src[(int64_t)(n0 + r) * w[l - 1] + k0 + lane]) : 0.f;
    __syncthreads();
    // layer 1 keeps the models side by side, [S][M * H1][Dp] and its
    // transpose; the others one matrix a model
    const bool one = l == 1;
    const int cn = one ? m * N + n0 : n0, KT = one ? pk.M * N : N;
    const size_t at = one ? (size_t)s * KT * K : sm * (size_t)N * K;
    float *f = (one ? dw.W1f : l == 2 ? dw.W2f : dw.W3f) + at, *ft = (one ? dw.W1Tf : l == 2 ? dw.W2Tf : dw.W3Tf) + at;
    const int r16 = lane & 15;
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // fragment (16 rows, 16 k): rows 16 wave, k 16 q
        const int n = wave * 16 + r16, k = q * 16 + (lane >> 4) * 4;
        *(float4*)(f + frag_index<float>(cn + n, k0 + k, K)) = make_float4(t[n][k], t[n][k + 1], t[n][k + 2], t[n][k + 3]);
        *(float4*)(ft + frag_index<float>(k0 + n, cn + k, KT)) = make_float4(t[k][n], t[k + 1][n], t[k + 2][n], t[k + 3][n]);
    }
    bf16_t *x = one ? dw.W1x : l == 2 ? dw.W2x : dw.W3x, *xt = one ? dw.W1Tx : l == 2 ? dw.W2Tx : dw.W3Tx;
    if (!x) return;
#pragma unroll
    for (int q = 0; q < 2; ++q) {   // fragment (16 rows, 32 k): rows 16 wave, k 32 q
        const int n = wave * 16 + r16, k = q * 32 + (lane >> 4) * 8;
        float v[8], vt[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = t[n][k + e];
            vt[e] = t[k + e][n];
        }
        uint4 o[kParts], ot[kParts];
        split8(v, o);
        split8(vt, ot);
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            *(uint4*)(x + kParts * at + split_index(cn + n, k0 + k, K) + 512 * p) = o[p];
            *(uint4*)(xt + kParts * at + split_index(k0 + n, cn + k, KT) + 512 * p) = ot[p];
        }
    }
}

template <typename TSRC>
hipError_t launch_set_nets(const TSRC* src, const ParamPack& pk, const DevWeights<PrecF32>& dw, hipStream_t st) {
    const int tiles = pk.H1 / 64 * (pk.Dp / 64) + pk.H2 / 64 * (pk.H1 / 64) + pk.H3 / 64 * (pk.H2 / 64);
    hipLaunchKernelGGL(k_set_nets<TSRC>, dim3(tiles + 1, pk.S * pk.M), dim3(256), 0, st, src, pk, dw);
    return hipGetLastError();
}
template hipError_t launch_set_nets<double>(const double*, const ParamPack&, const DevWeights<PrecF32>&, hipStream_t);
template hipError_t launch_set_nets<float>(const float*, const ParamPack&, const DevWeights<PrecF32>&, hipStream_t);

#define NNP_SETP(P, TSRC)                                                                          \
    template hipError_t launch_set_params<P, TSRC>(int64_t, int64_t, const TSRC*, const int32_t*,            \
                                                   const ParamPack&, const DevWeights<P>&, hipStream_t);
NNP_SETP(PrecF64, double)
NNP_SETP(PrecF64, float)
NNP_SETP(PrecF32, double)
NNP_SETP(PrecBF16, double)
NNP_SETP(PrecBF16, float)

}  // namespace nnp
