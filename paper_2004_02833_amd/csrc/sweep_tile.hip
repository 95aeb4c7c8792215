// Tile sweep: the forward substep with its source planes staged through LDS.
//
// A workgroup owns a box of W x TY x TZ cells (x, y, z; one cell per lane)
// and one pass of K target degrees, and walks the source columns mu = |m|
// upwards like the window sweep.  A stage is one (mu, cos or sin) column:
// its sources are the K + 1 degrees L0 - 1 + 2 b that exist, all on the same
// staggered grid, so all of them need the same one-sided neighbours.  Every
// source is copied to LDS as an image of the box's rows plus one halo row
// per z (y neighbour), one halo plane (z neighbour) and, where a row is cut
// into segments, one halo chunk per row (x neighbour), by 16-byte
// global-to-LDS copies that hold no registers; the next stage's images are
// in flight while a stage is computed.  Each source value is then requested
// from the caches (TY+1)(TZ+1)-1 / (TY TZ) times instead of three or four
// times per cell, and the registers this frees go into deeper passes, which
// re-read fewer shared source degrees.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "decay.h"
#include "kernels.h"

namespace pm {

namespace {

// 64 lanes x 16 bytes from base + voff (per lane) to LDS at ldsaddr + 16 lane.
// No register receives data; completion is waited for with vmcnt.  M0 is the
// LDS address.  It is a reserved register, which the compiler does not take in
// a clobber list and sets before uses of its own (indexed registers,
// messages); these kernels have none, so every s_mov to M0 in their code is
// this one.
__device__ __forceinline__ void copy16(uint32_t voff, uint64_t base, uint32_t ldsaddr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(base), "s"(ldsaddr)
                 : "memory");
}

__device__ __forceinline__ void wait_copies() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

constexpr int kXcd = 8;

template <class T, int K, int TPB, int QMAX, bool NT, bool ADJ, int WAVES>
__global__ void __launch_bounds__(TPB, WAVES)
k_sweep_tile(T* __restrict__ pool, StateOffs so, double* __restrict__ gp,
             const typename std::conditional<ADJ, double, T>::type* __restrict__ tab,
             const uint32_t* __restrict__ src, const uint32_t* __restrict__ tgt,
             const T* __restrict__ coef, double tau, int opening, int rowbase, int N, int parity,
             int npass, int per_xcd, TileGeom tg, GridDesc g) {
    using TabT = typename std::conditional<ADJ, double, T>::type;
    constexpr int E = 16 / (int)sizeof(T);
    constexpr int IMG = QMAX * 16;
    constexpr int BUF = (K + 1) * IMG;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * BUF];
    const int xcd = blockIdx.x % kXcd, j = blockIdx.x / kXcd;
    const int pass = npass - 1 - j / per_xcd, ti = j % per_xcd;
    const int bsz = tg.bx * tg.by * tg.bz;
    const int blk = (ti / bsz) * kXcd + xcd, in = ti % bsz;
    const int nbx = (tg.nseg + tg.bx - 1) / tg.bx, nby = (tg.nty + tg.by - 1) / tg.by;
    const int tx = (blk % nbx) * tg.bx + in % tg.bx;
    const int ty_ = (blk / nbx % nby) * tg.by + in / tg.bx % tg.by;
    const int tz_ = (blk / nbx / nby) * tg.bz + in / tg.bx / tg.by;
    if (pass < 0 || tx >= tg.nseg || ty_ >= tg.nty || tz_ >= tg.ntz) return;
    const int W = tg.w, TY = tg.ty, TZ = tg.tz;
    const int x0 = tx * W, y0 = ty_ * TY, z0 = tz_ * TZ;
    const int R = TY * TZ;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L0 = parity + 2 * K * pass;
    const int MU1 = N + 2;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int last = (int)(((g.ncell - 1) & ~(long long)(E - 1)) * (long long)sizeof(T));
    const int xf = x0 + W < nx ? x0 + W : 0, xb = x0 > 0 ? x0 - 1 : nx - 1;

    // ---- copy role: chunk tid of every image (row, chunk in the row)
    uint32_t offF = 0, offB = 0;
    int sel = 0;
    bool cp = false;
    {
        const int row = tid / tg.rowch, cc = tid - row * tg.rowch;
        int yf = y0, yb, zf = z0, zb;
        if (row < R) {
            yf = yb = y0 + row % TY;
            zf = zb = z0 + row / TY;
        } else if (row < R + TZ) {
            yf = y0 + TY;
            yb = y0 - 1 + ny;
            zf = zb = z0 + row - R;
            sel = 2;
        } else {
            yf = yb = y0 + max(0, (row - R - TZ)) % TY;
            zf = z0 + TZ;
            zb = z0 - 1 + nz;
            sel = 4;
        }
        cp = row < R + TZ + TY;
        const int rf = ((zf % nz) * ny + yf % ny) * nx, rb = ((zb % nz) * ny + yb % ny) * nx;
        int ef, eb;
        if (cc < tg.nmain) {
            ef = ((rf + x0) & ~(E - 1)) + cc * E;
            eb = ((rb + x0) & ~(E - 1)) + cc * E;
        } else {
            // the x neighbour outside the segment (the box's own rows only)
            cp = cp && row < R;
            sel = 1;
            ef = (rf + xf) & ~(E - 1);
            eb = (rf + xb) & ~(E - 1);
        }
        offF = min((uint32_t)ef * (uint32_t)sizeof(T), (uint32_t)last);
        offB = min((uint32_t)eb * (uint32_t)sizeof(T), (uint32_t)last);
    }
    // ---- cell role
    // (lanes past the box repeat its last row, unstored)
    const int lrow = min(tid / W, R - 1), lx = tid % W, ly = lrow % TY, lz = lrow / TY;
    const bool live = tid < W * R && x0 + lx < nx && y0 + ly < ny && z0 + lz < nz;
    const int rpe = tg.rowch * E;  // elements per row image
    uint32_t oc, oxx, oyy, ozz;    // byte offsets in an image: centre, x, y, z (forward | backward << 16)
    long long c;
    {
        auto rstart = [&](int y, int z) { return ((z % nz) * ny + y % ny) * nx; };
        auto elem = [&](int row, int y, int z) {  // element of this lane's x in a row image
            return row * rpe + ((rstart(y, z) + x0) & (E - 1)) + lx;
        };
        const int row = lrow, y = y0 + ly, z = z0 + lz;
        const int e = elem(row, y, z);
        oc = (uint32_t)e * (uint32_t)sizeof(T);
        int ep, em;
        if (tg.whole) {
            ep = lx + 1 == nx ? e - (nx - 1) : e + 1;
            em = lx == 0 ? e + (nx - 1) : e - 1;
        } else {
            const int hx = row * rpe + tg.nmain * E;
            ep = (lx == W - 1 || x0 + lx + 1 == nx) ? hx + ((rstart(y, z) + xf) & (E - 1)) : e + 1;
            em = lx == 0 ? hx + ((rstart(y, z) + xb) & (E - 1)) : e - 1;
        }
        if (ep < 0) ep = 0;
        if (lx >= nx) ep = em = e;
        oxx = (uint32_t)(ep * (int)sizeof(T)) | (uint32_t)(em * (int)sizeof(T)) << 16;
        ep = ly + 1 < TY ? elem(row + 1, y + 1, z) : elem(R + lz, y0 + TY, z);
        em = ly > 0 ? elem(row - 1, y - 1, z) : elem(R + lz, y0 - 1 + ny, z);
        oyy = (uint32_t)(ep * (int)sizeof(T)) | (uint32_t)(em * (int)sizeof(T)) << 16;
        ep = lz + 1 < TZ ? elem(row + TY, y, z + 1) : elem(R + TZ + ly, y, z0 + TZ);
        em = lz > 0 ? elem(row - TY, y, z - 1) : elem(R + TZ + ly, y, z0 - 1 + nz);
        ozz = (uint32_t)(ep * (int)sizeof(T)) | (uint32_t)(em * (int)sizeof(T)) << 16;
        c = ((long long)(z % nz) * ny + y % ny) * nx + min(x0 + lx, nx - 1);
    }

    const uint64_t sbase = (uint64_t)(uintptr_t)(pool + so.src);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds + wave * 1024;
    const int b1all = min(K + 1, (N - (L0 - 1)) / 2 + 1);
    const int t1 = min(K, (N - L0) / 2 + 1);
    auto bfirst = [&](int mu) { return mu > L0 - 1 ? (mu - L0 + 2) >> 1 : 0; };
    // staggering bits of every source of column (mu, ty)
    auto stag = [&](int mu, int ty) { return ((mu & 1) ^ ty) | ty << 1 | ((1 - parity + mu) & 1) << 2; };
    // Stream entries are plane offsets in units of 64 elements.
    constexpr int SH = sizeof(T) == 8 ? 9 : sizeof(T) == 4 ? 8 : 7;
    auto issue = [&](int mu, int ty) {
        if (ty == 1 && mu == 0) return;
        const uint32_t* sd = src + (((long long)pass * MU1 + mu) * 2 + ty) * (K + 1);
        const uint32_t voff = (stag(mu, ty) & sel) ? offB : offF;
        const int b0 = bfirst(mu);
        uint32_t sl[K + 1];
#pragma unroll
        for (int b = 0; b <= K; ++b) sl[b] = sd[b];
#pragma unroll
        for (int b = 0; b <= K; ++b) asm volatile("" ::"s"(sl[b]));
        if (cp) {
#pragma unroll
            for (int b = 0; b <= K; ++b)
                if (b >= b0 && b < b1all) copy16(voff, sbase + ((uint64_t)sl[b] << SH), lds0 + ty * BUF + b * IMG);
        }
    };
    issue(0, 0);

    const int mumax = min(N, L0 + 2 * (K - 1));
    // decay factors of the four target grids: [type][(mu + parity) mod 2]
    TabT fa[2][2], fb[2][2];
    auto trow = [&](int row) {
        return *(const TabT*)((const char*)(tab + (long long)row * g.ncell) + (uint32_t)c * (uint32_t)sizeof(TabT));
    };
#pragma unroll
    for (int ty = 0; ty < 2; ++ty)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            fa[ty][m] = trow(rowbase + 2 * (ty + 2 * m));
            fb[ty][m] = trow(rowbase + 2 * (ty + 2 * m) + 1);
            if (ADJ && opening) fa[ty][m] = fa[ty][m] * fa[ty][m] / ((TabT)1 + fa[ty][m]);
        }
    T S[3][K][2];
    T old[K][2];
    // transpose: the targets' values before and after the substep, and per
    // target grid [type][(mu + parity) mod 2] the sums of w u and w u', each
    // lane's own in LDS (in registers they spill)
    T pre[ADJ ? K : 1][2], post[ADJ ? K : 1][2];
    __shared__ double sums[ADJ ? 4 : 1][2][ADJ ? TPB : 1];
    if constexpr (ADJ) {
#pragma unroll
        for (int f = 0; f < 4; ++f) sums[f][0][tid] = sums[f][1][tid] = 0.0;
    }
    // (32-bit byte offsets: a plane has less than 2^31 bytes)
    auto grow = [&](int row) {
        return (double*)((char*)(gp + ((long long)pass * grad_rows(false) + row) * g.ncell) + (uint32_t)c * 8u);
    };
#pragma unroll
    for (int t = 0; t < K; ++t)
#pragma unroll
        for (int ty = 0; ty < 2; ++ty) {
            S[0][t][ty] = S[1][t][ty] = S[2][t][ty] = (T)0;
            old[t][ty] = (T)0;
            if constexpr (ADJ) pre[t][ty] = post[t][ty] = (T)0;
        }
    // Whole cache lines are streamed past the caches (nt); where rows start
    // inside a line, neighbouring segments share it and must meet in L2.
    auto load = [](const T* p) {
        if constexpr (NT)
            return __builtin_nontemporal_load(p);
        else
            return *p;
    };
    auto store = [](T v, T* p) {
        if constexpr (NT)
            __builtin_nontemporal_store(v, p);
        else
            *p = v;
    };
    const char* tin = (const char*)(pool + so.tin);
    char* tout = (char*)(pool + so.tout);
    const char* upre = (const char*)(pool + so.aux);
    const char* upost = (const char*)(pool + so.w);
    const uint32_t coff = (uint32_t)c * (uint32_t)sizeof(T);

    auto request = [&](int mu) {  // old values of target column mu
        const int t0 = mu > L0 ? (mu - L0 + 1) >> 1 : 0;
        const uint32_t* td = tgt + ((long long)pass * MU1 + mu) * 2 * K;
        uint32_t sl[2 * K];
#pragma unroll
        for (int t = 0; t < 2 * K; ++t) sl[t] = td[t];
#pragma unroll
        for (int t = 0; t < 2 * K; ++t) asm volatile("" ::"s"(sl[t]));
#pragma unroll
        for (int t = 0; t < K; ++t)
            if (t >= t0 && t < t1) {
                old[t][0] = load((const T*)(tin + ((uint64_t)sl[t] << SH) + coff));
                if (mu > 0) old[t][1] = load((const T*)(tin + ((uint64_t)sl[K + t] << SH) + coff));
                if constexpr (ADJ) {
                    pre[t][0] = load((const T*)(upre + ((uint64_t)sl[t] << SH) + coff));
                    post[t][0] = load((const T*)(upost + ((uint64_t)sl[t] << SH) + coff));
                    if (mu > 0) {
                        pre[t][1] = load((const T*)(upre + ((uint64_t)sl[K + t] << SH) + coff));
                        post[t][1] = load((const T*)(upost + ((uint64_t)sl[K + t] << SH) + coff));
                    }
                }
            }
    };
    auto update = [&](TabT a, TabT b, T u, T r) {  // r = q - S, transpose: S
        if constexpr (ADJ)
            return a * (double)u + b * (double)r;
        else if constexpr (std::is_same<T, double>::value)
            return a * u + b * r;
        else  // a = 1 - alpha
            return __builtin_fmaf(b, r, __builtin_fmaf(-a, u, u));
    };
    auto finish = [&](int mu) {  // column mu is complete in S[0]
        const int t0 = mu > L0 ? (mu - L0 + 1) >> 1 : 0;
        const uint32_t* td = tgt + ((long long)pass * MU1 + mu) * 2 * K;
        uint32_t sl[2 * K];
#pragma unroll
        for (int t = 0; t < 2 * K; ++t) sl[t] = td[t];
#pragma unroll
        for (int t = 0; t < 2 * K; ++t) asm volatile("" ::"s"(sl[t]));
        const bool m1 = (mu & 1) != parity;
        TabT al[2], be[2];
#pragma unroll
        for (int ty = 0; ty < 2; ++ty) {
            al[ty] = m1 ? fa[ty][1] : fa[ty][0];
            be[ty] = m1 ? fb[ty][1] : fb[ty][0];
        }
#pragma unroll
        for (int t = 0; t < K; ++t)
            if (t >= t0 && t < t1) {
                TabT a0 = al[0], b0 = be[0], q = (TabT)0;
                const bool mom0 = t == 0 && L0 == 0 && mu == 0;
                if (mom0) {
                    a0 = trow(kTabMom0);
                    b0 = trow(kTabMom0 + 1);
                    if constexpr (!ADJ) q = trow(kTabQ);
                    // arrived before the branch ends on every lane's path
                    asm volatile("" : "+v"(a0), "+v"(b0), "+v"(q));
                }
                const TabT v0 = update(a0, b0, old[t][0], ADJ ? S[0][t][0] : (T)(q - S[0][t][0]));
                const TabT v1 = update(al[1], be[1], old[t][1], ADJ ? S[0][t][1] : -S[0][t][1]);
                if constexpr (ADJ) {
                    if (mom0) {  // the one target of its set
                        if (live) *grow(8) += dl_dc(v0 * (double)pre[t][0], v0 * (double)post[t][0], a0, b0, tau);
                    } else {
                        sums[m1 ? 1 : 0][0][tid] += v0 * (double)pre[t][0];
                        sums[m1 ? 1 : 0][1][tid] += v0 * (double)post[t][0];
                    }
                    if (mu > 0) {
                        sums[m1 ? 3 : 2][0][tid] += v1 * (double)pre[t][1];
                        sums[m1 ? 3 : 2][1][tid] += v1 * (double)post[t][1];
                    }
                }
                if (live) {
                    store((T)v0, (T*)(tout + ((uint64_t)sl[t] << SH) + coff));
                    if (mu > 0) store((T)v1, (T*)(tout + ((uint64_t)sl[K + t] << SH) + coff));
                }
            }
    };
    // Sources in groups of G: their values and coefficients are requested
    // together (also for the empty slots of a group, unused) and waited for
    // once.
    constexpr int G = sizeof(T) == 8 ? 1 : 2;
    auto push = [&](int mu, auto TYC) {
        constexpr int ty = decltype(TYC)::value;
        const int b0 = bfirst(mu);
        const int bits = stag(mu, ty);
        const unsigned char* lc = lds + ty * BUF + oc;
        const unsigned char* lx_ = lds + ty * BUF + ((bits & 1) ? oxx >> 16 : oxx & 0xffffu);
        const unsigned char* ly_ = lds + ty * BUF + ((bits & 2) ? oyy >> 16 : oyy & 0xffffu);
        const unsigned char* lz_ = lds + ty * BUF + ((bits & 4) ? ozz >> 16 : ozz & 0xffffu);
        const T* cf = coef + (((long long)pass * MU1 + mu) * 2 + ty) * (K + 1) * 10;
#pragma unroll
        for (int g0 = 0; g0 <= K; g0 += G) {
            if (g0 + G <= b0 || g0 >= b1all) continue;
            T v[G], dx[G], dy[G], dz[G], kk[G][10];
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const int b = g0 + i;
                if (b > K) continue;
                v[i] = *(const T*)(lc + b * IMG);
                dx[i] = *(const T*)(lx_ + b * IMG);
                dy[i] = *(const T*)(ly_ + b * IMG);
                dz[i] = *(const T*)(lz_ + b * IMG);
#pragma unroll
                for (int r = 0; r < 10; ++r) kk[i][r] = cf[b * 10 + r];
            }
#pragma unroll
            for (int i = 0; i < G; ++i) {
                if (g0 + i > K) continue;
                asm volatile("" : "+v"(v[i]), "+v"(dx[i]), "+v"(dy[i]), "+v"(dz[i]));
                asm volatile("" ::"s"(kk[i][0]), "s"(kk[i][1]), "s"(kk[i][2]), "s"(kk[i][3]), "s"(kk[i][4]), "s"(kk[i][5]),
                             "s"(kk[i][6]), "s"(kk[i][7]), "s"(kk[i][8]), "s"(kk[i][9]));
            }
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const int b = g0 + i;
                if (b > K || b < b0 || b >= b1all) continue;
                const T ex = dx[i] - v[i], ey = dy[i] - v[i], ez = dz[i] - v[i];
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const int t = side == 0 ? b : b - 1;
                    if (t < 0 || t >= K) continue;
                    S[0][t][ty] += kk[i][side * 5] * ex;
                    S[0][t][1 - ty] += kk[i][side * 5 + 1] * ey;
                    S[1][t][ty] += kk[i][side * 5 + 2] * ez;
                    S[2][t][ty] += kk[i][side * 5 + 3] * ex;
                    S[2][t][1 - ty] += kk[i][side * 5 + 4] * ey;
                }
            }
        }
    };

    for (int mu = 0; mu <= mumax + 1; ++mu) {
        wait_copies();
        // the old target values have arrived too: taken here, so that no
        // later wait for them also waits for the copies issued below
#pragma unroll
        for (int t = 0; t < K; ++t) {
            asm volatile("" : "+v"(old[t][0]), "+v"(old[t][1]));
            if constexpr (ADJ) asm volatile("" : "+v"(pre[t][0]), "+v"(pre[t][1]), "+v"(post[t][0]), "+v"(post[t][1]));
        }
        __syncthreads();
        issue(mu, 1);
        if (mu >= 2) finish(mu - 2);
        if (mu >= 1) {
            request(mu - 1);
#pragma unroll
            for (int t = 0; t < K; ++t)
#pragma unroll
                for (int ty = 0; ty < 2; ++ty) {
                    S[0][t][ty] = S[1][t][ty];
                    S[1][t][ty] = S[2][t][ty];
                    S[2][t][ty] = (T)0;
                }
        }
        push(mu, std::integral_constant<int, 0>());
        wait_copies();
        __syncthreads();
        if (mu <= mumax) issue(mu + 1, 0);
        if (mu > 0) push(mu, std::integral_constant<int, 1>());
    }
    finish(mumax);
    if constexpr (ADJ) {
        // dL/dc of the parity's grids (row = grid in storage order); one
        // workgroup owns every (pass, cell)
        if (live) {
#pragma unroll
            for (int ty = 0; ty < 2; ++ty)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int f = ty + 2 * m;
                    *grow((parity ? 4 : 0) + f) +=
                        dl_dc(sums[2 * ty + m][0][tid], sums[2 * ty + m][1][tid], trow(rowbase + 2 * f), fb[ty][m], tau);
                }
        }
    }
}

template <class T, int K, int TPB, int QMAX, bool NT, bool ADJ, int WAVES = 4>
void launch_t(void* pool, StateOffs so, double* gp, const void* tab, double tau, int opening, int rowbase, const TileArgs& a, const TileGeom& tg, const GridDesc& g, hipStream_t st) {
    const int nblk = ((tg.nseg + tg.bx - 1) / tg.bx) * ((tg.nty + tg.by - 1) / tg.by) * ((tg.ntz + tg.bz - 1) / tg.bz);
    const int per_xcd = (nblk + kXcd - 1) / kXcd * tg.bx * tg.by * tg.bz;
    using TabT = typename std::conditional<ADJ, double, T>::type;
    hipLaunchKernelGGL((k_sweep_tile<T, K, TPB, QMAX, NT, ADJ, WAVES>), dim3((unsigned)(kXcd * per_xcd * a.npass)), dim3(TPB), 0, st, (T*)pool,
                       so, gp, (const TabT*)tab, a.src, a.tgt, (const T*)a.coef, tau, opening, rowbase, a.N, a.parity, a.npass,
                       per_xcd, tg, g);
}

}  // namespace

// Workgroup size: two workgroups of 512 fill a CU's registers at 128 each;
// one of 1024 with boxes twice as large was slower (P39 64^3 odd sweep FP64
// 1.03 vs 0.95 ms, FP32 0.51 vs 0.50).
constexpr int kTpb = 512;
// Largest image in 16-byte chunks: 2 (K + 1) of them per workgroup, two
// workgroups (FP64) or three (FP32, K = 4) in 160 KB.
constexpr int kQ64 = 476, kQ32 = 264;

// Box shape for a grid.  Memory traffic decides, idle lanes matter little,
// so the cost of a shape is the product of
//   the halo requests it adds per cell, weighted by how often they miss L2
//   (a z neighbour's box is further away in time than a y neighbour's),
//   a quarter of the lanes it leaves idle, and
//   a penalty for short contiguous runs; rows that start inside a cache line
//   cost more, and cutting rows of whole lines inside a line is excluded.
// Measured odd sweeps: P39 64^3 FP64 64x2x4 0.949, 64x4x2 0.971, 32x4x4
// 1.033 ms; P39 80x80x40 FP64 80x2x3 1.079, 80x3x2 1.128, 40x4x3 1.281; P9
// 100x75x50 FP64 50x5x2 0.128, 100x2x2 0.136, 64x2x4 0.144; P39 160^3 FP32
// 32x4x4 8.88, 64x2x4 8.85, 40x4x3 (cut inside lines) 14.9 ms.
bool tile_geom(int prec, const GridDesc& g, TileGeom& tg) {
    if (prec != kF64 && prec != kF32) return false;
    const int esz = prec == kF64 ? 8 : 4, E = 16 / esz;
    if (g.pstride * esz >= (1LL << 31)) return false;  // 32-bit byte offsets in a plane
    const int qmax = prec == kF64 ? kQ64 : kQ32;
    const bool al = g.nx % E == 0;
    const bool rows_fit = g.nx * (long long)esz % 128 == 0;
    double best = 1e30;
    for (int nseg = 1; nseg <= (g.nx + 15) / 16; ++nseg) {
        const int W = ((g.nx + nseg - 1) / nseg + E - 1) / E * E;
        if (W > kTpb || (nseg - 1) * W >= g.nx) continue;
        const bool whole = nseg == 1;
        if (rows_fit && !whole && W * esz % 128) continue;
        const int nmain = W / E + (al ? 0 : 1), rowch = nmain + (whole ? 0 : 1);
        for (int TY = 1; TY * W <= kTpb; ++TY)
            for (int TZ = 1; TZ * TY * W <= kTpb; ++TZ) {
                const int rows = TY * TZ + TY + TZ;
                if (rows * rowch > qmax || rows * rowch > kTpb) continue;
                const int nty = (g.ny + TY - 1) / TY, ntz = (g.nz + TZ - 1) / TZ;
                const double util = (double)g.ncell / ((double)nseg * nty * ntz * kTpb);
                const double halo = 0.3 / TY + 0.5 / TZ + (whole ? 0.0 : 0.3 * 64 / (W * esz));
                const double run = (double)W * esz * (whole ? TY : 1);
                const double cost = (1.0 + halo) * (0.75 + 0.25 / util) * (1.0 + (rows_fit ? 45.0 : 70.0) / run);
                if (cost < best) {
                    best = cost;
                    tg = TileGeom{W, TY, TZ, nseg, nty, ntz, rowch, nmain, whole ? 1 : 0, 1, 1, 1};
                }
            }
    }
    if (best > 1e29) return false;
    // Blocks of boxes go round the XCDs: neighbours in a block share halo
    // rows in one L2, and the eight XCDs work next to each other in every
    // plane (contiguous eighths of the grid per XCD: P39 160^3 FP64 18.3 vs
    // 17.0 ms, 64^3 0.968 vs 0.943).  The largest block that spreads the
    // boxes within 2% of evenly, at most 64 boxes, or 16 and two in y where
    // the grid has many (160^3 FP64: blocks of 5 / 20 / 80 boxes 16.9 / 17.2 /
    // 18.0 ms; FP32 5x1x2 / 5x2x2 / 5x4x1 8.68 / 8.75 / 8.80; P19 250^3 FP32
    // 3x1x2 / 3x2x2 / 3x4x1 9.65 / 9.64 / 9.97).  More than eight segments go
    // in the blocks of five to eight that leave the fewest empty places: 9 as
    // 8 + 1 gave every other XCD one box to eight (P12 540x40x40 FP64 604 us
    // a sweep, as 5 + 4 457; window 469).
    tg.bx = tg.nseg < 8 ? tg.nseg : 8;
    for (int b = 7; tg.nseg > 8 && b >= 5; --b)
        if ((tg.nseg + b - 1) / b * b < (tg.nseg + tg.bx - 1) / tg.bx * tg.bx) tg.bx = b;
    const long long nbox = (long long)tg.nseg * tg.nty * tg.ntz;
    const int cap = nbox > 1024 ? 16 : 64;
    double most = 1e30;
    int size = 0;
    for (int bz = 8; bz >= 1; bz /= 2)
        for (int by = nbox > 1024 ? 2 : 8; by >= 1; by /= 2) {
            const int n = tg.bx * by * bz;
            if (n > cap && by * bz > 1) continue;
            const long long nblk = (long long)((tg.nseg + tg.bx - 1) / tg.bx) * ((tg.nty + by - 1) / by) * ((tg.ntz + bz - 1) / bz);
            double uneven = (double)((nblk + kXcd - 1) / kXcd * kXcd * n) / (double)nbox;
            if (uneven < 1.02) uneven = 1.0;
            if (uneven < most - 1e-9 || (uneven < most + 1e-9 && n > size)) {
                most = uneven;
                size = n;
                tg.by = by;
                tg.bz = bz;
            }
        }
    return true;
}

// Target degrees per pass for `nd` target degrees: as few passes as the
// registers allow (128 at two workgroups per CU: 4 degrees in FP64), evenly
// filled.  P39 160^3 FP64 18.3 / 17.6 / 17.1 ms at 2 / 3 / 4.  FP32 goes
// to 5: 64^3 is the same at 4 / 5 / 8 / 10 (0.503 / 0.512 / 0.526 / 0.502 ms;
// deeper passes re-read less but keep fewer workgroups in flight), larger
// grids gain (P39 160^3 8.57 vs 8.45 ms at 4 / 5, P19 250^3 9.53 vs 9.19, P25
// 97x60x133 0.828 vs 0.755).
// The transpose holds three values per target: 2 degrees in FP64, 4 in FP32.
// Contexts have nd >= 3 (P5 on), so FP64 passes take 3 or 4.
int tile_depth(int prec, int nd, bool adj) {
    if (adj) return prec == kF64 ? 2 : 4;
    const int kmax = prec == kF64 ? 4 : 5;
    const int np = (nd + kmax - 1) / kmax, want = (nd + np - 1) / np;
    return prec == kF64 ? want : want <= 4 ? 4 : 5;
}

// Whether the tile sweep runs a context that the low-order sweep does not take
// (FP64 from P5, FP32 from P8 on).  Measured per sweep, window / tile in us:
// - It needs enough workgroups (boxes x passes) to fill the chip with boxes of
//   512 cells; the window sweep's smaller groups win below (FP64 240: P7 48^3
//   27.0 / 30.9, 432: P19 48x40x36 90.7 / 79.8; FP32 768: P19 64x64x48 99 /
//   109, 900: P19 60^3 116 / 129, 960: P39 48^3 368 / 243).
// - Boxes with most lanes idle copy more padding than values: rows of one
//   cell, half the lanes idle and more (FP64 P7 1x512x512 53 / 79, 1x1x400000
//   78 / 388; FP32 P12 2x512x512 110 / 261), FP32 up to 0.7 of them busy (P12
//   5x300x300 0.71 of the window's speed, 5x600x600 0.84).
// - FP32 rows of up to 64 cells are contiguous in the window sweep's linear
//   tiles, and on planes that start on cache lines its chunks are whole lines;
//   there the tile sweep gains only from 3072 boxes on, or as many workgroups
//   from P14 on (P12 20x130x97 0.91, P19 33x90x61 0.80, 56^3 0.76 of its
//   speed, 40x200x200 1.03 and 1.13; P9 96^3 0.87, 66x128x100 0.79,
//   66x200x200 1.13).  Rows of 16, 32 and 48 cells and boxes with their lanes
//   filled stay (P12 48x80x80 1.79, 128x64x64 1.11).
// - Ten odd degrees are three FP64 passes, 4 + 4 + 2: with 257 to 344 boxes the
//   first two run over the 512 workgroups that fit at a time and the rest
//   cannot fill a second round (P19 36x60x60, 270 boxes, 0.92 of the window's
//   speed, 50x50x56, 280, 0.89, 30x70x70, 324, 0.92; 50^3, 250, 1.04 and
//   56^3, 361, 1.01; P18 and P21 gain there).
// - Rows longer than 64 cells with fewer than four planes leave three of four
//   window waves idle (P12 512x512x1 2.5 times the window's speed).
bool tile_use(int prec, int N, const GridDesc& g, TileGeom& tg) {
    if (N < 5 || !tile_geom(prec, g, tg)) return false;  // P0 comes here too: no dual moments
    const int nd = N / 2 + 1, K = tile_depth(prec, nd, false);
    const long long boxes = (long long)tg.nseg * tg.nty * tg.ntz, nwg = boxes * ((nd + K - 1) / K);
    const double util = (double)g.ncell / ((double)boxes * kTpb);
    if (nwg < (prec == kF64 ? 320 : 950) || util <= 0.5) return false;
    if (prec == kF64) return !((N + 1) / 2 == 10 && boxes > 256 && boxes < 345 && g.nx <= 64);
    if (g.nz < 4 && g.nx > 64) return true;
    if (util < 0.7) return false;
    const bool few = boxes < 3072 && (N < 14 || nwg < 3072);
    if (few && g.nx < 64 && g.nx % 16) return false;
    const bool planes_on_lines = (long long)g.nx * g.ny * 4 % 128 == 0;
    return !(few && N < 14 && util < 0.8 && planes_on_lines);
}

// Whether the transpose of a low-order context above P4 (where that sweep has
// none) runs as a tile sweep, and not as a window sweep.  Whole reverse passes,
// window / tile: FP64 gains where the window's accesses are short or cross
// rows, from 320 boxes on (P5 64^3 1.13, 161x45x33 1.14, P6 32x80x80 1.13; but P5
// 56^3 0.95, 33x90x61 0.96).  FP32 runs four degrees in one pass, so
// the boxes must fill their rounds of 512 (P7 128x64x64, 1024 boxes, 1.43, 60^3,
// 450, 1.12, 97x60x133, 2010, 1.26; 20x130x97, 520, 0.85, 33x130x111, 1064,
// 0.93), with most lanes busy (P5 5x200x200 0.84).
bool tile_use_adj(int prec, int N, const GridDesc& g, TileGeom& tg) {
    if (N <= kLowAdjMax || !tile_geom(prec, g, tg)) return false;
    const long long boxes = (long long)tg.nseg * tg.nty * tg.ntz;
    const double util = (double)g.ncell / ((double)boxes * kTpb);
    if (prec == kF64) return boxes >= 320 && util > 0.5 && (g.nx % 16 == 0 || g.nx > 64);
    const int nd = N / 2 + 1, K = tile_depth(prec, nd, true);
    const long long nwg = boxes * ((nd + K - 1) / K);
    return util > 0.7 && (double)nwg >= 0.7 * (double)((nwg + 511) / 512 * 512);
}

hipError_t tile_load() {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, (const void*)k_sweep_tile<double, 4, kTpb, kQ64, true, false, 4>);
}

static bool whole_lines(int prec, const TileGeom& tg, const GridDesc& g) {
    const long long esz = prec == kF64 ? 8 : 4;
    return g.nx * esz % 128 == 0 && (tg.whole || tg.w * esz % 128 == 0);
}

hipError_t launch_sweep_tile(int prec, void* pool, StateOffs so, const double* tab, const float* tabf, int rowbase, const TileArgs& a,
                             const TileGeom& tg, const GridDesc& g, hipStream_t st) {
    const bool nt = whole_lines(prec, tg, g);
    const void* tb = prec == kF64 ? (const void*)tab : (const void*)tabf;
#define PM_TILE(T, KK, Q)                                                                                        \
    case KK:                                                                                                     \
        if (nt)                                                                                                  \
            launch_t<T, KK, kTpb, Q, true, false>(pool, so, nullptr, tb, 0.0, 0, rowbase, a, tg, g, st);         \
        else                                                                                                     \
            launch_t<T, KK, kTpb, Q, false, false>(pool, so, nullptr, tb, 0.0, 0, rowbase, a, tg, g, st);        \
        break;
    // FP32 at depth 5 on large grids: held to 80 registers (two spilled),
    // three workgroups fit a CU instead of two (P39 160^3 8.45 vs 8.66 ms, P19
    // 250^3 9.19 vs 9.64); with fewer workgroups than four rounds of that, two
    // run as well without the spills (P39 64^3 504 vs 497 us).
    if (prec == kF32 && a.K == 5 && (long long)tg.nseg * tg.nty * tg.ntz * a.npass >= 3072) {
        if (nt)
            launch_t<float, 5, kTpb, kQ32, true, false, 6>(pool, so, nullptr, tb, 0.0, 0, rowbase, a, tg, g, st);
        else
            launch_t<float, 5, kTpb, kQ32, false, false, 6>(pool, so, nullptr, tb, 0.0, 0, rowbase, a, tg, g, st);
        return hipGetLastError();
    }
    if (prec == kF64) {
        switch (a.K) {
            PM_TILE(double, 3, kQ64)
            PM_TILE(double, 4, kQ64)
            default: return hipErrorInvalidValue;
        }
    } else if (prec == kF32) {
        switch (a.K) {
            PM_TILE(float, 4, kQ32)
            PM_TILE(float, 5, kQ32)
            default: return hipErrorInvalidValue;
        }
    } else {
        return hipErrorInvalidValue;
    }
#undef PM_TILE
    return hipGetLastError();
}

hipError_t launch_adj_tile(int prec, void* pool, StateOffs so, double* gp, const double* tab, int rowbase, double tau, int opening,
                           const TileArgs& a, const TileGeom& tg, const GridDesc& g, hipStream_t st) {
    const bool nt = whole_lines(prec, tg, g);
#define PM_TILE(T, KK, Q)                                                                                        \
    if (nt)                                                                                                      \
        launch_t<T, KK, kTpb, Q, true, true>(pool, so, gp, tab, tau, opening, rowbase, a, tg, g, st);            \
    else                                                                                                         \
        launch_t<T, KK, kTpb, Q, false, true>(pool, so, gp, tab, tau, opening, rowbase, a, tg, g, st);
    if (prec == kF64 && a.K == 2) {
        PM_TILE(double, 2, kQ64)
    } else if (prec == kF32 && a.K == 4) {
        PM_TILE(float, 4, kQ32)
    } else {
        return hipErrorInvalidValue;
    }
#undef PM_TILE
    return hipGetLastError();
}

}  // namespace pm
