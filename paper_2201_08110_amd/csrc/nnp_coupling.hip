// nnp_coupling.hip -- the NNP-MM coupling term of an NNP/MM step.
//
// Mechanical embedding (Methods, Eq. 4): every NNP atom i interacts with
// every MM atom j through a Coulomb term k q_i q_j / r and a 12-6
// Lennard-Jones term 4 eps_ij ((sigma_ij/r)^12 - (sigma_ij/r)^6), with
// Lorentz-Berthelot pair parameters sigma_ij = (sigma_i + sigma_j)/2,
// eps_ij = sqrt(eps_i eps_j) and an optional plain cutoff.  Forces act on both
// sides.  Both force sums are formed without atomics and in a fixed order:
//
// k_couple_pairs evaluates every pair once.  A wave takes 16 MM atoms at a
// time against 64 NNP atoms (staged in LDS): row r of 16 lanes holds the same
// 16 MM atoms and NNP atoms 16 r .. 16 r + 15, lane c meeting atom (c + t) mod
// 16 in step t.  The MM force stays in its lane; the NNP force sums move one
// lane along the row a step (a DPP rotation), so after 16 steps each is back in
// its atom's lane.  Each workgroup writes partial F_i and E; k_couple_sum adds
// them in a fixed order.
//
// 64 x 47,648 pairs, FP32: evaluating each pair once per side took 12.1 + 5.4 us,
// this 8.6 + 2.5.  Bound by vector ALU issue (about 45 instructions a pair) and
// the latency of one trip through memory.  Summing in the same launch (the last
// workgroup of 16 sums theirs, the last of those the rest) took 18.2: each of
// the two hand-overs waits for memory three times.
#include <algorithm>

#include <hip/hip_runtime.h>

#include "nnp_internal.h"

namespace nnp {

// per-atom operands staged in LDS: x, y, z, q, sigma/2, sqrt(eps)
constexpr int kCoupleVals = 6;
constexpr int kCoupleThreads = 1024, kCoupleWaves = kCoupleThreads / 64;

template <typename T> __device__ inline T c_rsqrt(T x);
template <> __device__ inline float c_rsqrt<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <> __device__ inline double c_rsqrt<double>(double x) { return 1.0 / sqrt(x); }

// energy of the pair and (dV/dr)/r
template <typename T>
__device__ inline void couple_pair(T k, T r2, T qq, T sig, T se, T& v, T& dvr) {
    const T ri = c_rsqrt(r2);
    const T ri2 = ri * ri;
    const T coul = k * qq * ri;
    const T s2 = sig * sig * ri2;
    const T s6 = s2 * s2 * s2, s12 = s6 * s6;
    const T e4 = T(4) * se;   // 4 eps_ij
    v = coul + e4 * (s12 - s6);
    dvr = (-coul - e4 * (T(12) * s12 - T(6) * s6)) * ri2;
}

template <typename T>
__device__ inline void load_atom(const T* __restrict__ x, const T* __restrict__ par, int i, T out[kCoupleVals]) {
    out[0] = x[3 * (size_t)i];
    out[1] = x[3 * (size_t)i + 1];
    out[2] = x[3 * (size_t)i + 2];
    out[3] = par[3 * (size_t)i];
    out[4] = T(0.5) * par[3 * (size_t)i + 1];
    out[5] = sqrt(par[3 * (size_t)i + 2]);
}

// v from the next lane of its row of 16 (the last from the first)
__device__ inline float row_next(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x12f, 0xf, 0xf, false));   // row_ror:15
}
__device__ inline double row_next(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x12f, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x12f, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sums: an MM atom's force in T over 64 NNP atoms (four partial sums of 16), the
// 64s in order, and once onto the caller's; an NNP atom's in T over 16 MM atoms
// and in FP64 beyond, the energy in FP64.
// A wave goes through kCoupleRounds of its groups block by block of 64 NNP
// atoms, so the sums of a block leave the waves once for them all; between
// blocks the groups' MM forces wait in LDS.
// With few groups, `share` waves (a power of two) deal a group's blocks out among
// themselves and meet in LDS: a wave's chain is one block instead of all (1,024
// x 100 pairs 55.5 -> 13.6 us in FP32, 65 x 3,000 in FP64 13.4 -> 10.3).
// KIND: at most 64 NNP atoms (one block), more of them, or more of them shared.
constexpr int kCoupleRounds = 8;
enum { COUPLE_ONE = 0, COUPLE_MANY = 1, COUPLE_SHARED = 2 };
template <typename T> size_t couple_lds(int n_nnp) {
    const size_t np = (size_t)(std::max(n_nnp, 1) + 63) / 64 * 64;
    return sizeof(T) * kCoupleVals * np +
           (np > 64 ? sizeof(double) * 3 * np + sizeof(T) * 48 * kCoupleWaves * kCoupleRounds : 0);
}
template <typename T, bool CUT, int KIND>
__global__ __launch_bounds__(kCoupleThreads) void k_couple_pairs(int n_nnp, const T* __restrict__ x_nnp,
                                                                 const T* __restrict__ par_nnp, int n_mm,
                                                                 const T* __restrict__ x_mm,
                                                                 const T* __restrict__ par_mm, T k, T rc2,
                                                                 T* __restrict__ F_mm, int accumulate, int share,
                                                                 double* __restrict__ e_part,
                                                                 T* __restrict__ f_part) {
    constexpr bool MANY = KIND != COUPLE_ONE;
    extern __shared__ __align__(16) char smem[];
    __shared__ double red[kCoupleWaves][3][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15;
    const int P = KIND == COUPLE_SHARED ? share : 1, slots = kCoupleWaves / P;
    const int slot = wave / P, first = wave % P;   // this wave's place among the groups and blocks
    const int ngroups = (n_mm + 15) / 16, nw = gridDim.x * slots;
    const int g0 = slot * gridDim.x + blockIdx.x;      // consecutive groups go to different workgroups
    if (n_nnp == 0) {
        for (int i = blockIdx.x * kCoupleThreads + tid; !accumulate && i < 3 * n_mm; i += gridDim.x * kCoupleThreads)
            F_mm[i] = T(0);
        if (tid == 0) e_part[blockIdx.x] = 0.0;
        return;
    }
    T b[kCoupleVals] = {0, 0, 0, 0, 0, 0};
    if (g0 < ngroups) load_atom(x_mm, par_mm, min(g0 * 16 + c, n_mm - 1), b);   // in flight while the NNP atoms are staged
    // [6][np], past n_nnp the last atom again without charge, size and well
    // depth: its pairs are finite wherever that atom's are
    const int nblk = MANY ? (n_nnp + 63) / 64 : 1, np = nblk * 64;
    T* s = (T*)smem;
    double* tot = (double*)(s + kCoupleVals * np);     // [3][np] this workgroup's NNP forces
    T* keep = (T*)(tot + 3 * np) + wave * 48 * kCoupleRounds;   // [round][3][16]
    for (int i = tid; i < np; i += kCoupleThreads) {
        T a[kCoupleVals];
        load_atom(x_nnp, par_nnp, min(i, n_nnp - 1), a);
        if (i >= n_nnp) a[3] = a[4] = a[5] = T(0);
#pragma unroll
        for (int v = 0; v < kCoupleVals; ++v) s[v * np + i] = a[v];
    }
    for (int i = tid; MANY && i < 3 * np; i += kCoupleThreads) tot[i] = 0.0;
    __syncthreads();
    double e = 0.0;
    const int step = MANY ? kCoupleRounds * nw : ngroups;
    for (int gs = 0; gs < ngroups; gs += step) {
        const int ge = min(gs + step, ngroups);
        for (int b0 = 0; b0 < nblk; b0 += P) {
            const int blk = b0 + first;
            const T* sb = s + blk * 64 + (lane & 48);
            double fi[3] = {0.0, 0.0, 0.0};
            T* kp = keep;
            for (int g = gs + g0; blk < nblk && g < ge; g += nw, kp += 48) {
                const int j = g * 16 + c;
                const bool act = j < n_mm;
                if (g != g0 || b0 > 0) load_atom(x_mm, par_mm, act ? j : n_mm - 1, b);
                if (!act) b[3] = b[5] = T(0);          // no charge, no well depth: no force, no energy
                T fj[3] = {0, 0, 0}, fr[3] = {0, 0, 0};
#pragma unroll 4
                for (int t = 0; t < 16; ++t) {
                    const T* q = sb + ((c + t) & 15);
                    const T d0 = b[0] - q[0], d1 = b[1] - q[np], d2 = b[2] - q[2 * np];
                    const T r2 = d0 * d0 + d1 * d1 + d2 * d2;
                    // a pair beyond the cutoff takes no part: with an atom at
                    // infinity, zero times its distance would not be zero
                    if (!CUT || !(r2 >= rc2)) {
                        T v, dvr;
                        couple_pair(k, r2, q[3 * np] * b[3], q[4 * np] + b[4], q[5 * np] * b[5], v, dvr);
                        e += (double)v;
                        // F_i = -dV/dx_i = (dV/dr) d / r, F_j = -F_i
                        fj[0] -= dvr * d0;
                        fj[1] -= dvr * d1;
                        fj[2] -= dvr * d2;
                        fr[0] += dvr * d0;
                        fr[1] += dvr * d1;
                        fr[2] += dvr * d2;
                    }
#pragma unroll
                    for (int d = 0; d < 3; ++d) fr[d] = row_next(fr[d]);
                }
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    fi[d] += (double)fr[d];
                    fj[d] += __shfl_xor(fj[d], 16);
                    fj[d] += __shfl_xor(fj[d], 32);
                }
                if (MANY && lane < 16) {
                    if (b0 > 0)
#pragma unroll
                        for (int d = 0; d < 3; ++d) fj[d] = kp[16 * d + c] + fj[d];
                    if (P > 1 || blk + 1 < nblk)
#pragma unroll
                        for (int d = 0; d < 3; ++d) kp[16 * d + c] = fj[d];
                }
                if (act && lane < 16 && P == 1 && blk + 1 == nblk) {
                    T* F = F_mm + 3 * (size_t)j;
#pragma unroll
                    for (int d = 0; d < 3; ++d) F[d] = (accumulate ? F[d] : T(0)) + fj[d];
                }
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) red[wave][d][lane] = fi[d];
            __syncthreads();
            for (int q = wave / 3; q < P && q < nblk - b0; q += kCoupleWaves / 3) {   // block b0 + q
                if (wave >= kCoupleWaves / 3 * 3) break;
                const int d = wave % 3;
                double v = 0.0;
                for (int w = 0; w < slots; ++w) v += red[w * P + q][d][lane];
                if (MANY) tot[d * np + (b0 + q) * 64 + lane] += v;
                else if (lane < n_nnp) f_part[(size_t)(3 * lane + d) * gridDim.x + blockIdx.x] = (T)v;
            }
            __syncthreads();
        }
        if (MANY && P > 1 && first == 0 && lane < 16) {
            // (the waves' sums are behind the last barrier; one round: share
            // > 1 comes with a slot a group)
            const int g = gs + g0, j = g * 16 + c;
            if (g < ge && j < n_mm) {
                T* F = F_mm + 3 * (size_t)j;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    T v = keep[16 * d + c];
                    for (int q = 1; q < P && q < nblk; ++q) v += keep[q * 48 * kCoupleRounds + 16 * d + c];
                    F[d] = (accumulate ? F[d] : T(0)) + v;
                }
            }
        }
    }
    for (int i = tid; MANY && i < 3 * n_nnp; i += kCoupleThreads)
        f_part[(size_t)i * gridDim.x + blockIdx.x] = (T)tot[i % 3 * np + i / 3];
    for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o);
    if (lane == 0) red[wave][0][0] = e;
    __syncthreads();
    if (tid == 0) {
        double v = 0.0;
        for (int w = 0; w < kCoupleWaves; ++w) v += red[w][0][0];
        e_part[blockIdx.x] = v;
    }
}

// One workgroup per NNP force component (and one for the energy), one partial
// a thread, then a fixed tree, so the sum is the same on every run.
template <typename T>
__global__ __launch_bounds__(kCoupleMaxWg) void k_couple_sum(int n_nnp, int n, const T* __restrict__ f_part,
                                                             const double* __restrict__ e_part,
                                                             T* __restrict__ F_nnp, double* __restrict__ E,
                                                             int accumulate) {
    __shared__ double red[kCoupleMaxWg / 64];
    const int t = blockIdx.x, w = threadIdx.x;   // component (t < 3 n_nnp) or the energy
    const bool energy = t == 3 * n_nnp;
    double v = w >= n ? 0.0 : energy ? e_part[w] : (double)f_part[(size_t)t * n + w];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((w & 63) == 0) red[w >> 6] = v;
    __syncthreads();
    if (w > 0) return;
    v = (red[0] + red[1]) + (red[2] + red[3]);
    if (energy) *E = accumulate ? *E + v : v;
    else F_nnp[t] = accumulate ? F_nnp[t] + (T)v : (T)v;
}

template <typename T, bool CUT> auto couple_kernel(int n_nnp, int share) {
    return n_nnp <= 64 ? k_couple_pairs<T, CUT, COUPLE_ONE>
           : share > 1 ? k_couple_pairs<T, CUT, COUPLE_SHARED>
                       : k_couple_pairs<T, CUT, COUPLE_MANY>;
}

// bytes of the partials of a call with n_nnp NNP atoms
size_t coupling_scratch_bytes(int n_nnp, size_t tsz) {
    return kCoupleMaxWg * (sizeof(double) + tsz * 3 * (size_t)n_nnp);
}

template <typename T>
hipError_t launch_coupling(const CouplingShape& cs, int n_nnp, const T* x_nnp, const T* par_nnp,
                           int n_mm, const T* x_mm, const T* par_mm, double* E, T* F_nnp, T* F_mm,
                           void* scratch, bool accumulate, hipStream_t st) {
    const T k = (T)cs.coulomb_k, rc2 = (T)(cs.cutoff > 0 ? cs.cutoff * cs.cutoff : 0.0);
    double* e_part = (double*)scratch;
    T* f_part = (T*)(e_part + kCoupleMaxWg);
    // one workgroup per CU at most, and four busy waves a workgroup at least:
    // few groups of 16 MM atoms spread over many CUs.  A group's blocks of 64
    // NNP atoms are shared while every group has its waves at the same time
    const int ng = (n_mm + 15) / 16, nblk = (n_nnp + 63) / 64;
    int share = 1;
    while (share < kCoupleWaves && share < nblk && ng * 2 * share <= kCoupleMaxWg * kCoupleWaves) share *= 2;
    const int per = std::max(4 / share, 1), nwg = std::min(kCoupleMaxWg, (ng + per - 1) / per);
    if (nwg > 0) {
        const size_t lds = couple_lds<T>(n_nnp);
        auto kern = rc2 > T(0) ? couple_kernel<T, true>(n_nnp, share) : couple_kernel<T, false>(n_nnp, share);
        hipError_t e = ensure_lds((const void*)kern, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(nwg), dim3(kCoupleThreads), lds, st, n_nnp, x_nnp, par_nnp, n_mm, x_mm, par_mm,
                           k, rc2, F_mm, accumulate ? 1 : 0, share, e_part, f_part);
    }
    hipLaunchKernelGGL(k_couple_sum<T>, dim3(3 * n_nnp + 1), dim3(kCoupleMaxWg), 0, st, n_nnp, nwg, f_part,
                       e_part, F_nnp, E, accumulate ? 1 : 0);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scratch of the allocation-free coupling entry point: the per-block energy
// partials and the per-chunk NNP force partials live in this array instead
// of a handle's workspace.  Every GPU the library runs on holds its own copy
// for the lifetime of the process; host code uses only the device address
// obtained below, never the array's name.
static __device__ __align__(256) unsigned char scratch[kCoupleScratchBytes];

hipError_t coupling_scratch(void** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        // raise the pair kernel's dynamic-LDS limit now (its largest size),
        // so later calls do no host-side set-up
        const auto raise = [&](auto zero) {
            typedef decltype(zero) T;
            for (const auto& kern : {couple_kernel<T, false>(64, 1), couple_kernel<T, true>(64, 1)})
                if (e == hipSuccess) e = ensure_lds((const void*)kern, couple_lds<T>(64));
            for (int share : {1, 2})
                for (const auto& kern : {couple_kernel<T, false>(1024, share), couple_kernel<T, true>(1024, share)})
                    if (e == hipSuccess) e = ensure_lds((const void*)kern, couple_lds<T>(1024));
        };
        raise(float());
        raise(double());
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

template hipError_t launch_coupling<float>(const CouplingShape&, int, const float*, const float*, int,
                                           const float*, const float*, double*, float*, float*, void*, bool,
                                           hipStream_t);
template hipError_t launch_coupling<double>(const CouplingShape&, int, const double*, const double*,
                                            int, const double*, const double*, double*, double*, double*, void*,
                                            bool, hipStream_t);

}  // namespace nnp
