// Low-order sweep: the forward substep of orders N <= kLowMax with nothing
// left to a loop.  A lane owns one cell, requests every source value and its
// one-sided x, y and z neighbours, every old target value and its decay
// factors at once, and forms all targets of the parity: one memory latency
// per sweep, where the column loop of the other sweeps waits once per column.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "decay.h"
#include "kernels.h"

namespace pm {

namespace {

struct B16 {
    uint16_t b;
};
typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ double val(double v) { return v; }
__device__ __forceinline__ float val(float v) { return v; }
__device__ __forceinline__ float val(B16 v) { return __uint_as_float((uint32_t)v.b << 16); }
__device__ __forceinline__ void put(double& o, double v) { o = v; }
__device__ __forceinline__ void put(float& o, float v) { o = v; }
__device__ __forceinline__ void put(B16& o, float v) {
    const f32x2 p = {v, 0.0f};
    o.b = (uint16_t)(__builtin_bit_cast(uint32_t, __builtin_convertvector(p, b16x2)) & 0xffffu);
}

// Moments of one parity before degree l, and the place of (l, mu, type) in
// its degree (mu = 0 first, then cos and sin of each mu).
constexpr int before(int l) { return l * (l - 1) / 2; }
constexpr int place(int mu, int ty) { return mu == 0 ? 0 : 2 * mu - 1 + ty; }

constexpr int kXcd = 8;

// Target degrees per pass: all of them up to N = 7; above, where only small
// grids come here, two (the last pass the two highest), to spread the work.
constexpr int passes(int N, int par) {
    const int nd = (N - par) / 2 + 1;
    return N <= 7 ? 1 : (nd + 1) / 2;
}
constexpr int first_degree(int N, int par, int pass) {
    const int nd = (N - par) / 2 + 1;
    const int i = nd - 2 * (passes(N, par) - pass);
    return par + 2 * (N <= 7 || i < 0 ? 0 : i);
}
constexpr int end_degree(int N, int par, int pass) {  // past the last one
    return pass + 1 < passes(N, par) ? first_degree(N, par, pass + 1) : N + 1;
}

// Factors and update in FP64 for FP64 storage and the transpose, else FP32.
template <class T, bool ADJ>
using TabOf = typename std::conditional<ADJ || std::is_same<T, double>::value, double, float>::type;

// Targets of degrees LA, LA + 2, .. below LB of cell c; ADJ: one transposed
// substep (see the modes of the window sweep), gp the pass's gradient rows.
template <class T, int N, int PAR, int LA, int LB, bool NT, bool ADJ>
__device__ __forceinline__ void low_pass(T* __restrict__ pool, const StateOffs& so, double* __restrict__ gp,
                                         const TabOf<T, ADJ>* __restrict__ tab, double tau, int opening, int rowbase,
                                         const LowArgs& a, uint32_t c, const GridDesc& g) {
    using F = TabOf<T, ADJ>;
    using A = typename std::conditional<std::is_same<T, double>::value, double, float>::type;
    constexpr int SA = LA > 0 ? LA - 1 : 1;                       // source degrees SA .. SB
    constexpr int LL = LA + (LB - 1 - LA) / 2 * 2;                // last target degree
    constexpr int SB = LL + 1 <= N ? LL + 1 : LL - 1;
    constexpr int S0 = before(SA), NS = before(SB + 2) - S0;
    constexpr int T0 = before(LA), NTG = before(LL + 2) - T0;
    const uint32_t nx = g.nx, ny = g.ny, nz = g.nz;
    const uint32_t row = c / nx, x = c - row * nx, z = row / ny, y = row - z * ny;
    const int xp = x + 1 == nx ? 1 - (int)nx : 1, xm = x == 0 ? (int)nx - 1 : -1;
    const int yp = (y + 1 == ny ? 1 - (int)ny : 1) * (int)nx, ym = (y == 0 ? (int)ny - 1 : -1) * (int)nx;
    const long long nxy = (long long)nx * ny;
    const long long zp = (z + 1 == nz ? 1 - (int)nz : 1) * nxy, zm = (z == 0 ? (int)nz - 1 : -1) * nxy;

    T rc[NS > 0 ? NS : 1], rx[NS > 0 ? NS : 1], ry[NS > 0 ? NS : 1], rz[NS > 0 ? NS : 1];
#pragma unroll
    for (int l = SA; l <= SB; l += 2)
#pragma unroll
        for (int k = 0; k < 2 * N + 1; ++k) {
            if (k >= 2 * l + 1) continue;
            const int mu = (k + 1) / 2, ty = k == 0 ? 0 : (k + 1) % 2;
            const int s = before(l) + k - S0;
            const T* p = pool + so.src + (long long)a.src[s + S0] * 64 + c;
            rc[s] = p[0];
            rx[s] = p[((mu & 1) ^ ty) ? xm : xp];
            ry[s] = p[ty ? ym : yp];
            rz[s] = p[((l + mu) & 1) ? zm : zp];
        }
    T old[NTG];
#pragma unroll
    for (int t = 0; t < NTG; ++t) {
        const T* p = pool + so.tin + (long long)a.tgt[t + T0] * 64 + c;
        if constexpr (NT && !std::is_same<T, B16>::value)
            old[t] = __builtin_nontemporal_load(p);
        else
            old[t] = *p;
    }
    F fa[4], fb[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        fa[f] = tab[(long long)(rowbase + 2 * f) * g.ncell + c];
        fb[f] = tab[(long long)(rowbase + 2 * f + 1) * g.ncell + c];
    }
    F a0 = 0, b0 = 0, q = 0;
    if constexpr (LA == 0) {
        a0 = tab[(long long)kTabMom0 * g.ncell + c];
        b0 = tab[(long long)(kTabMom0 + 1) * g.ncell + c];
        if constexpr (!ADJ) q = tab[(long long)kTabQ * g.ncell + c];
    }
    A S[NTG];
#pragma unroll
    for (int t = 0; t < NTG; ++t) S[t] = 0;
    const A* coef = (const A*)a.coef;
#pragma unroll
    for (int l = SA; l <= SB; l += 2)
#pragma unroll
        for (int k = 0; k < 2 * N + 1; ++k) {
            if (k >= 2 * l + 1) continue;
            const int mu = (k + 1) / 2, ty = k == 0 ? 0 : (k + 1) % 2;
            const int s = before(l) + k - S0;
            const A v = val(rc[s]);
            const A dx = val(rx[s]) - v, dy = val(ry[s]) - v, dz = val(rz[s]) - v;
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int lt = side == 0 ? l + 1 : l - 1;
                if (lt < LA || lt > LL) continue;
                const int b = before(lt) - T0;
                const A* kk = coef + ((s + S0) * 2 + side) * 5;
                // the five couplings of a source: x and y to mu - 1, z, x and y to mu + 1
                if (mu >= 1 && mu - 1 <= lt && !(mu == 1 && ty == 1)) S[b + place(mu - 1, ty)] += kk[0] * dx;
                if (mu >= 1 && mu - 1 <= lt && !(mu == 1 && ty == 0)) S[b + place(mu - 1, 1 - ty)] += kk[1] * dy;
                if (mu <= lt) S[b + place(mu, ty)] += kk[2] * dz;
                if (mu + 1 <= lt) S[b + place(mu + 1, ty)] += kk[3] * dx;
                if (mu + 1 <= lt) S[b + place(mu + 1, 1 - ty)] += kk[4] * dy;
            }
        }
    T pre[ADJ ? NTG : 1], post[ADJ ? NTG : 1];
    if constexpr (ADJ) {
        // requested once the sources are used up: all at once they overflow
        // the registers
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < NTG; ++t) {
            pre[t] = pool[so.aux + (long long)a.tgt[t + T0] * 64 + c];
            post[t] = pool[so.w + (long long)a.tgt[t + T0] * 64 + c];
        }
    }
    double gA[5] = {0, 0, 0, 0, 0}, gB[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int l = LA; l <= LL; l += 2)
#pragma unroll
        for (int k = 0; k < 2 * N + 1; ++k) {
            if (k >= 2 * l + 1) continue;
            const int mu = (k + 1) / 2, ty = k == 0 ? 0 : (k + 1) % 2;
            const int t = before(l) + k - T0;
            const int f = ty + 2 * ((mu & 1) ^ PAR);  // target grid within the parity
            const F al = l == 0 ? a0 : fa[f], be = l == 0 ? b0 : fb[f];
            F v;
            if constexpr (ADJ) {
                const double m = opening ? al * al / (1.0 + al) : al;
                v = m * (double)val(old[t]) + be * (double)S[t];
                const int set = l == 0 ? 4 : f;
                gA[set] += v * (double)val(pre[t]);
                gB[set] += v * (double)val(post[t]);
            } else {
                const A r = (l == 0 ? q : (F)0) - S[t];
                const A u = val(old[t]);
                if constexpr (std::is_same<T, double>::value)
                    v = al * u + be * r;
                else  // al = 1 - alpha
                    v = __builtin_fmaf(be, r, __builtin_fmaf(-al, u, u));
            }
            T o;
            put(o, v);
            T* p = pool + so.tout + (long long)a.tgt[t + T0] * 64 + c;
            if constexpr (NT && !std::is_same<T, B16>::value)
                __builtin_nontemporal_store(o, p);
            else
                *p = o;
        }
    if constexpr (ADJ) {
        // dL/dc of the parity's grids; one lane owns every (pass, cell)
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            if (f == 4 && LA > 0) continue;
            gp[(long long)(f == 4 ? 8 : (PAR ? 4 : 0) + f) * g.ncell + c] +=
                dl_dc(gA[f], gB[f], f == 4 ? a0 : fa[f & 3], f == 4 ? b0 : fb[f & 3], tau);
        }
    }
}

template <class T, int N, int PAR, bool NT, bool ADJ>
__global__ void __launch_bounds__(256)
k_sweep_low(T* __restrict__ pool, StateOffs so, double* __restrict__ gp, const TabOf<T, ADJ>* __restrict__ tab, double tau,
            int opening, int rowbase, LowArgs a, int group, GridDesc g) {
    constexpr int NP = passes(N, PAR);
    // groups of consecutive workgroups on one XCD (neighbour rows meet in its
    // L2), the passes of a workgroup's cells back to back
    const uint32_t xcd = blockIdx.x % kXcd, j = blockIdx.x / kXcd / NP, pass = NP - 1 - blockIdx.x / kXcd % NP;
    const uint32_t blk = ((j / group) * kXcd + xcd) * group + j % group;
    const uint32_t c = blk * blockDim.x + threadIdx.x;
    if (c >= (uint32_t)g.ncell) return;
#define PM_LOW_PASS(P)                                                                                                            \
    if constexpr (P < NP)                                                                                                         \
        if (pass == P)                                                                                                            \
            low_pass<T, N, PAR, first_degree(N, PAR, P), end_degree(N, PAR, P), NT, ADJ>(                                         \
                pool, so, gp + (long long)P * grad_rows(false) * g.ncell, tab, tau, opening, rowbase, a, c, g);
    PM_LOW_PASS(0)
    PM_LOW_PASS(1)
    PM_LOW_PASS(2)
#undef PM_LOW_PASS
}

struct LowCall {
    void* pool;
    StateOffs so;
    double* gp;
    const void* tab;
    double tau;
    int opening, rowbase;
    const LowArgs& a;
    const GridDesc& g;
    hipStream_t st;
};

template <class T, int N, int PAR, bool ADJ>
void launch_p(const LowCall& k) {
    const int tpb = k.g.ncell < 262144 ? 64 : 256;
    const long long nblk = (k.g.ncell + tpb - 1) / tpb;
    const int group = (int)(nblk < 1024 ? (nblk + kXcd - 1) / kXcd : 128);
    const long long ngroup = (nblk + group - 1) / group;
    const unsigned nwg = (unsigned)((ngroup + kXcd - 1) / kXcd * kXcd * group * passes(N, PAR));
    // targets streamed past the caches only where the state does not fit them
    const bool nt = (long long)(N + 1) * (N + 1) * k.g.pstride * (long long)sizeof(T) > (128LL << 20);
    if (nt && !ADJ)
        hipLaunchKernelGGL((k_sweep_low<T, N, PAR, !ADJ, ADJ>), dim3(nwg), dim3(tpb), 0, k.st, (T*)k.pool, k.so, k.gp,
                           (const TabOf<T, ADJ>*)k.tab, k.tau, k.opening, k.rowbase, k.a, group, k.g);
    else
        hipLaunchKernelGGL((k_sweep_low<T, N, PAR, false, ADJ>), dim3(nwg), dim3(tpb), 0, k.st, (T*)k.pool, k.so, k.gp,
                           (const TabOf<T, ADJ>*)k.tab, k.tau, k.opening, k.rowbase, k.a, group, k.g);
}

template <class T, int N, bool ADJ>
hipError_t launch_n(int parity, const LowCall& k) {
    if constexpr (ADJ && N > kLowAdjMax) {
        return hipErrorInvalidValue;
    } else {
        if (parity)
            launch_p<T, N, 1, ADJ>(k);
        else
            launch_p<T, N, 0, ADJ>(k);
        return hipGetLastError();
    }
}

template <class T, bool ADJ>
hipError_t launch_t(int N, int parity, const LowCall& k) {
    switch (N) {
        case 1: return launch_n<T, 1, ADJ>(parity, k);
        case 2: return launch_n<T, 2, ADJ>(parity, k);
        case 3: return launch_n<T, 3, ADJ>(parity, k);
        case 4: return launch_n<T, 4, ADJ>(parity, k);
        case 5: return launch_n<T, 5, ADJ>(parity, k);
        case 6: return launch_n<T, 6, ADJ>(parity, k);
        case 7: return launch_n<T, 7, ADJ>(parity, k);
        case 8: return launch_n<T, 8, ADJ>(parity, k);
        case 9: return launch_n<T, 9, ADJ>(parity, k);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

int low_passes(int N, int parity) { return passes(N, parity); }

// The code of a source file is loaded when one of its kernels is first used:
// 4.4 ms inside the first step (P7 64^3 FP32; 0.08 ms with this call),
// which may also be under stream capture.  Asking for a kernel's attributes
// loads it while the context is made.
hipError_t low_load() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, (const void*)k_sweep_low<double, 1, 0, false, false>);
}

// Whether the low-order sweep runs a grid of ncell cells: always where the
// sources of a cell fit the registers of two waves per SIMD, else on grids
// small enough for latency to decide.  Measured per sweep against the faster
// of the other two: FP64 P4 160x150x170 302 vs 313 us, P5 64^3 23.0 vs 26.5
// and 128^3 218 vs 212, P6 60^3 29.4 vs 32.2 and 75^3 64.5 vs 56.5, P7 48^3
// 21.5 vs 26.8 and 64^3 45.7 vs 41.6, P8 32^3 13.0 vs 20.6 and 57x41x35 37 vs
// 28; FP32 P7 128^3 170 vs 178, P8 57x41x35 17 vs 22 and 128^3 322 vs 235, P9
// 32^3 10.9 vs 18.4 and 57x41x35 26 vs 24; BF16 P6 128^3 75 vs 94, P7 90^3 37
// vs 63 and 128^3 124 vs 108, P8 64^3 20.8 vs 27.7, P9 57x41x35 19.0 vs 20.2.
bool low_use(int prec, int N, long long ncell) {
    if (N < 1 || N > kLowMax) return false;
    if (N == 9) return ncell <= 40000;
    if (prec == kF64) return N <= 4 || ncell <= (N <= 6 ? 300000 : N == 7 ? 120000 : 40000);
    if (prec == kF32) return N <= 7 || ncell <= 100000;
    return N <= 6 || ncell <= (N == 7 ? 1000000 : 300000);
}

hipError_t launch_sweep_low(int prec, int N, int parity, void* pool, StateOffs so, const double* tab, const float* tabf, int rowbase,
                            const LowArgs& a, const GridDesc& g, hipStream_t st) {
    const LowCall k{pool, so, nullptr, prec == kF64 ? (const void*)tab : (const void*)tabf, 0.0, 0, rowbase, a, g, st};
    if (prec == kF64) return launch_t<double, false>(N, parity, k);
    if (prec == kF32) return launch_t<float, false>(N, parity, k);
    return launch_t<B16, false>(N, parity, k);
}

hipError_t launch_adj_low(int prec, int N, int parity, void* pool, StateOffs so, double* gp, const double* tab, int rowbase, double tau,
                          int opening, const LowArgs& a, const GridDesc& g, hipStream_t st) {
    const LowCall k{pool, so, gp, tab, tau, opening, rowbase, a, g, st};
    if (prec == kF64) return launch_t<double, true>(N, parity, k);
    if (prec == kF32) return launch_t<float, true>(N, parity, k);
    return hipErrorInvalidValue;
}

}  // namespace pm
