// C ABI of libpm: context management, validation and the step driver.
//
// A time step is the Strang composition of eq. (6): the odd-grid half step,
// the even-grid full step and the odd-grid half step, each one sweep launch
// on the bound stream (paper Sec. 2.1 and Sec. 3.2, where a step is the
// sweeps S^o, S^e, S^o).  The gradient pass walks the recorded steps
// backwards from device checkpoints (the paper has no derivatives; this is
// the transpose of the discrete step).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <utility>
#include <vector>

#include "../../include/pm.h"
#include "kernels.h"
#include "pm_internal.h"

namespace {

std::string g_err = "no error";
int g_pending_prec = PM_FP64;
std::vector<double> g_pending_scat;  // g_1, g_2, ... for the next pm_init
int g_merge = 1;
hipStream_t g_bound = nullptr;  // caller's stream (nullptr: own stream)

int fail(int code, const std::string& msg) {
    g_err = msg;
    return code;
}

#define HIPCHK(x)                                                                   \
    do {                                                                            \
        hipError_t e_ = (x);                                                        \
        if (e_ != hipSuccess)                                                       \
            return fail(e_ == hipErrorOutOfMemory ? PM_ENOMEM : PM_EDEVICE,         \
                        std::string(#x) + ": " + hipGetErrorString(e_));            \
    } while (0)

size_t elem_size(int prec) { return prec == PM_FP64 ? 8 : prec == PM_FP32 ? 4 : 2; }

// Halo faces of the sweeps of one parity (see halo_plan).
struct HaloPlan {
    std::vector<int> slots;  // slots of the faces' moments, face after face
    pm::HaloFaces hf{};
};

struct Ctx {
    bool live = false;
    int dev = -1;  // device of its memory and stream
    int N = 0, V = 0, nx = 0, ny = 0, nz = 0;
    long long ncell = 0;
    double h[3] = {0, 0, 0};  // cell edges dx, dy, dz
    double dt = 0;
    int prec = PM_FP64;
    size_t esz = 8;
    pm::GridDesc g{};
    pm::Layout L;
    long long ve = 0;  // planes of the even parity (slots [0, ve)); odd ones follow
    void* u = nullptr;
    double* tab = nullptr;
    float* tabf = nullptr;  // float copy for the FP32 update (float/bfloat16 storage, isotropic)
    double* sig = nullptr;  // sigma_a, sigma_s on the device, until the tables are made
    bool aniso = false;     // some g_l != 0 for 1 <= l <= N
    double* gl = nullptr;   // g_0 .. g_N on the device (anisotropic scattering)
    void* win_mem = nullptr;  // window sweep streams (both parities)
    HaloPlan halo[2];         // halo faces of the sweeps of each parity
    int* halo_slots[2] = {nullptr, nullptr};
    void* adj_mem = nullptr;  // streams of the transposed sweeps when their depth differs
    pm::WinArgs win[2]{};     // forward sweeps
    pm::WinArgs wadj[2]{};    // transposed sweeps (pm_grad)
    bool tiled = false;       // forward sweeps run as tile sweeps
    bool tiled_adj = false;   // and the transposed ones
    pm::TileGeom tg{};
    pm::TileArgs tile[2]{}, tadj[2]{};  // forward and transposed
    void* tile_mem[2] = {nullptr, nullptr};
    bool low = false;         // forward sweeps run as low-order sweeps
    bool low_adj = false;     // and the transposed ones
    pm::LowArgs lowa[2]{};
    void* low_mem = nullptr;
    double* plane64 = nullptr;
    double* red = nullptr;
    unsigned long long* redc = nullptr;
    int npart = 256;   // partial sums of pm_total (its rounding depends on it)
    int ncheck = 1024; // partial results of pm_check / pm_check_noalloc
    hipStream_t own = nullptr;
    int cfl_warn = 0;
    int ck = 0;
    long long rec_steps = 0;
    std::vector<void*> ckpts;
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[2];
    long long dev_bytes = 0;
    long long base_bytes = 0;

    size_t state_bytes() const { return (size_t)V * (size_t)g.pstride * esz; }
    // element offset of the first plane of a parity within a state
    long long half(int parity) const { return parity ? ve * g.pstride : 0; }
    int passes(int parity) const {
        return low ? pm::low_passes(N, parity) : tiled ? tile[parity].npass : win[parity].npass;
    }
    int adj_passes(int parity) const {
        return low_adj ? pm::low_passes(N, parity) : tiled_adj ? tadj[parity].npass : wadj[parity].npass;
    }
    hipStream_t stream() const { return g_bound ? g_bound : own; }
    void* plane(void* base, int slot) const {
        return (char*)base + (size_t)slot * (size_t)g.pstride * esz;
    }
};

Ctx C;

// Device memory.  Freed blocks are kept for the next allocation of about
// their size on the same device: a program that fits a medium builds a
// context, records and differentiates over and over, and gigabytes returned
// to the driver are wiped before it hands them out again (P7 64^3, 100
// recorded steps: a forward and gradient 41 ms on a fresh device, 140 ms
// after large contexts).  While a context is replaced its blocks wait for the
// new one; afterwards at most 1/32 of the device's memory stays, and at most
// 1/8 of what is free there, since other users of the card cannot ask for it;
// all of it is given back when an allocation fails here and by pm_finalize, and
// the checks of free memory count it as free.
struct Block {
    void* p;
    size_t bytes;
    int dev;
};
std::vector<Block> g_used, g_kept;  // g_kept: the longest kept first
constexpr size_t kKeptBlocks = 256;  // searched one by one

int this_device() {
    int d = 0;
    (void)hipGetDevice(&d);
    return d;
}

// Gives kept blocks back until at most `most` bytes in kKeptBlocks blocks
// stay: those that are larger by themselves, then the longest kept, so that
// what a repeated call has just freed is there for the next one.
void trim_kept(size_t most) {
    size_t sum = 0, n = g_kept.size();
    for (Block& b : g_kept)
        if (b.bytes > most) {
            (void)hipFree(b.p);
            b.p = nullptr;
            --n;
        } else {
            sum += b.bytes;
        }
    for (Block& b : g_kept) {
        if (sum <= most && n <= kKeptBlocks) break;
        if (!b.p) continue;
        (void)hipFree(b.p);
        b.p = nullptr;
        sum -= b.bytes;
        --n;
    }
    g_kept.erase(std::remove_if(g_kept.begin(), g_kept.end(), [](const Block& b) { return !b.p; }), g_kept.end());
}

// hipMemGetInfo with the kept blocks of this device counted as free.
hipError_t free_memory(size_t* fr, size_t* total = nullptr) {
    size_t tot = 0;
    const hipError_t e = hipMemGetInfo(fr, &tot);
    const int dev = this_device();
    if (e == hipSuccess)
        for (const Block& b : g_kept)
            if (b.dev == dev) *fr += b.bytes;
    if (total) *total = tot;
    return e;
}

void trim_kept_to_share() {
    size_t fr = 0, tot = 0;
    if (!g_kept.empty() && free_memory(&fr, &tot) == hipSuccess) trim_kept(std::min(tot / 32, fr / 8));
}

template <class P>
int dmalloc(P** p, size_t bytes, const char* what) {
    const int dev = this_device();
    const size_t want = bytes ? bytes : 1;
    auto best = g_kept.end();
    for (auto it = g_kept.begin(); it != g_kept.end(); ++it)
        if (it->dev == dev && it->bytes >= want && it->bytes <= want + want / 8 + 4096 &&
            (best == g_kept.end() || it->bytes < best->bytes))
            best = it;
    Block b{nullptr, want, dev};
    if (best != g_kept.end()) {
        b = *best;
        g_kept.erase(best);
    } else {
        hipError_t e = hipMalloc(&b.p, want);
        if (e != hipSuccess && !g_kept.empty()) {
            (void)hipGetLastError();
            trim_kept(0);
            e = hipMalloc(&b.p, want);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(e == hipErrorOutOfMemory ? PM_ENOMEM : PM_EDEVICE,
                        std::string("hipMalloc(") + what + ", " + std::to_string(bytes) +
                            " bytes): " + hipGetErrorString(e));
        }
    }
    g_used.push_back(b);
    C.dev_bytes += (long long)bytes;
    *p = (P*)b.p;
    return PM_OK;
}

// The caller has waited for the work that uses the block (wait_context: as
// hipFree would).
void dfree(void* p) {
    if (!p) return;
    for (size_t i = g_used.size(); i-- > 0;)
        if (g_used[i].p == p) {
            g_kept.push_back(g_used[i]);
            g_used.erase(g_used.begin() + (long)i);
            return;
        }
}

// Waits for everything queued on the context's device, which need not be the
// current one.
void wait_context() {
    const int dev = this_device();
    const bool other = C.dev >= 0 && C.dev != dev;
    if (other) (void)hipSetDevice(C.dev);
    (void)hipDeviceSynchronize();
    if (other) (void)hipSetDevice(dev);
}

// The library's own stream, kept from context to context on a device.
hipStream_t g_own = nullptr;
int g_own_dev = -1;

hipError_t own_stream(hipStream_t* s) {
    const int dev = this_device();
    if (g_own && g_own_dev != dev) {
        (void)hipStreamDestroy(g_own);
        g_own = nullptr;
    }
    if (!g_own) {
        const hipError_t e = hipStreamCreate(&g_own);
        if (e != hipSuccess) {
            g_own = nullptr;
            return e;
        }
        g_own_dev = dev;
    }
    *s = g_own;
    return hipSuccess;
}

// Identifies the recorded forward: changes whenever the recording starts,
// stops, is dropped or is extended by pm_step (pm_recording_id).
long long g_rec_id = 1;

void drop_recording(bool replacing = false) {
    if (!C.ckpts.empty()) {
        if (!replacing) wait_context();
        for (void* p : C.ckpts) dfree(p);
        C.ckpts.clear();
        if (!replacing) trim_kept_to_share();
    }
    C.rec_steps = 0;
    ++g_rec_id;
}

void drop_events() {
    for (auto& v : C.ev)
        for (auto& pr : v) {
            (void)hipEventDestroy(pr.first);
            (void)hipEventDestroy(pr.second);
        }
    C.ev[0].clear();
    C.ev[1].clear();
}

void release() {
    if (C.u || C.tab) wait_context();
    drop_recording(true);
    drop_events();
    dfree(C.u);
    dfree(C.tab);
    dfree(C.tabf);
    dfree(C.sig);
    dfree(C.gl);
    dfree(C.win_mem);
    dfree(C.tile_mem[0]);
    dfree(C.tile_mem[1]);
    dfree(C.low_mem);
    dfree(C.halo_slots[0]);
    dfree(C.halo_slots[1]);
    dfree(C.adj_mem);
    dfree(C.plane64);
    dfree(C.red);
    dfree(C.redc);
    C = Ctx();
}

bool finite_nonneg(const double* a, long long n, const char* name, std::string& msg) {
    for (long long i = 0; i < n; ++i)
        if (!std::isfinite(a[i]) || a[i] < 0.0) {
            msg = std::string(name) + "[" + std::to_string(i) + "] is negative or not finite";
            return false;
        }
    return true;
}

// Plane stride: a multiple of 64 elements, padded so that consecutive planes
// do not sit at power-of-two distances.
long long plane_stride(long long ncell) {
    long long s = (ncell + 63) / 64 * 64;
    if ((s & (s - 1)) == 0 && s >= 4096) s += 64;
    return s;
}

// The flux entries by target row (at most ten each).
struct FluxRows {
    std::vector<pm::FluxEntry> e;
    std::vector<int> begin;
    long long nnz_par[2] = {0, 0};  // entries with targets of a parity

    explicit FluxRows(int N) : begin((size_t)(N + 1) * (N + 1) + 1, 0) {
        const std::vector<pm::FluxEntry> all = pm::flux_entries(N);
        for (const pm::FluxEntry& f : all) ++begin[f.row + 1];
        for (size_t i = 1; i < begin.size(); ++i) begin[i] += begin[i - 1];
        e.resize(all.size());
        std::vector<int> at(begin.begin(), begin.end() - 1);
        for (const pm::FluxEntry& f : all) e[at[f.row]++] = f;
        for (int l = 0; l <= N; ++l) nnz_par[l & 1] += begin[(size_t)(l + 1) * (l + 1)] - begin[(size_t)l * l];
    }
    const double* find(int row, int col, int dir) const {
        for (int k = begin[row]; k < begin[row + 1]; ++k)
            if (e[k].col == col && e[k].dir == dir) return &e[k].val;
        return nullptr;
    }
};

// Streams of the window sweep (layout documented in kernels.h).  Every
// nonzero flux entry with a target of the sweep's parity must land in exactly
// one coefficient slot; the count is checked.
int build_window_tables(int K, pm::WinArgs (&win)[2], void** mem) {
    const pm::Layout& L = C.L;
    // columns mu = 0..N+1 and one empty column N+2: a sweep requests the next
    // column's sources unconditionally
    const int N = C.N, V = C.V, MU1 = N + 3;
    const FluxRows flux(N);
    const long long* nnz_par = flux.nnz_par;
    auto exists = [&](int l, int mu, int ty) {
        return l >= 0 && l <= N && mu >= 0 && mu <= l && !(ty == 1 && mu == 0);
    };
    auto idx = [](int l, int mu, int ty) { return l * l + l + (ty == 0 ? mu : -mu); };
    struct Host {
        std::vector<int2> src, tgt;
        std::vector<double> coef;
    } H[2];
    for (int p = 0; p < 2; ++p) {
        const int npass = N >= p ? (N - p) / (2 * K) + 1 : 0;
        win[p].N = N;
        win[p].parity = p;
        win[p].K = K;
        win[p].npass = npass;
        Host& h = H[p];
        h.src.assign((size_t)npass * MU1 * (K + 1) * 2, make_int2(-1, 0));
        h.tgt.assign((size_t)npass * MU1 * K * 2, make_int2(-1, 0));
        h.coef.assign((size_t)npass * MU1 * (K + 1) * 20, 0.0);
        long long used = 0;
        for (int pass = 0; pass < npass; ++pass) {
            const int L0 = p + 2 * K * pass;
            for (int mu = 0; mu < MU1; ++mu) {
                for (int b = 0; b <= K; ++b)
                    for (int ty = 0; ty < 2; ++ty) {
                        const int ls = L0 - 1 + 2 * b;
                        if (!exists(ls, mu, ty)) continue;
                        const int j = idx(ls, mu, ty);
                        const int bits = pm::grid_bits(ls, ty == 0 ? mu : -mu);
                        h.src[((size_t)(pass * MU1 + mu) * (K + 1) + b) * 2 + ty] =
                            make_int2(L.slot_of[j] - (p ? 0 : (int)C.ve), bits);
                        for (int side = 0; side < 2; ++side) {
                            const int t = side == 0 ? b : b - 1;
                            if (t < 0 || t >= K) continue;
                            const int lt = L0 + 2 * t;
                            // (target column, target type, direction) of the five roles
                            const int tmu[5] = {mu - 1, mu - 1, mu, mu + 1, mu + 1};
                            const int tty[5] = {ty, 1 - ty, ty, ty, 1 - ty};
                            const int dir[5] = {0, 1, 2, 0, 1};
                            for (int r = 0; r < 5; ++r) {
                                if (!exists(lt, tmu[r], tty[r])) continue;
                                const int i = idx(lt, tmu[r], tty[r]);
                                const double* val = flux.find(i, j, dir[r]);
                                if (!val) continue;
                                const double sgn = ((bits >> dir[r]) & 1) ? -1.0 : 1.0;
                                h.coef[((((size_t)(pass * MU1 + mu) * (K + 1) + b) * 2 + ty) * 2 + side) * 5 + r] =
                                    sgn * *val / C.h[dir[r]];
                                ++used;
                            }
                        }
                    }
                for (int t = 0; t < K; ++t)
                    for (int ty = 0; ty < 2; ++ty) {
                        const int lt = L0 + 2 * t;
                        if (!exists(lt, mu, ty)) continue;
                        const int i = idx(lt, mu, ty);
                        const int row = i == 0 ? pm::kTabMom0 : 2 * L.order_of[i];
                        h.tgt[((size_t)(pass * MU1 + mu) * K + t) * 2 + ty] =
                            make_int2(L.slot_of[i] - (p ? (int)C.ve : 0), row);
                    }
            }
        }
        if (used != nnz_par[p])
            return fail(PM_EINVAL, "internal: window streams cover " + std::to_string(used) + " of " +
                                       std::to_string(nnz_par[p]) + " couplings");
        // slots count from the first plane of their parity half
        const long long nhalf[2] = {C.ve, (long long)V - C.ve};
        for (const int2& e : h.src)
            if (e.x >= nhalf[1 - p]) return fail(PM_EINVAL, "internal: source slot outside its half");
        for (const int2& e : h.tgt)
            if (e.x >= nhalf[p]) return fail(PM_EINVAL, "internal: target slot outside its half");
    }
    const bool f64 = C.prec == PM_FP64;
    const size_t es = f64 ? sizeof(double) : sizeof(float);
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    size_t total = 0, off[2][3];
    for (int p = 0; p < 2; ++p) {
        off[p][0] = total; total += up(H[p].src.size() * sizeof(int2));
        off[p][1] = total; total += up(H[p].tgt.size() * sizeof(int2));
        off[p][2] = total; total += up(H[p].coef.size() * es);
    }
    int rc = dmalloc(mem, total, "window streams");
    if (rc) return rc;
    char* base = (char*)*mem;
    for (int p = 0; p < 2; ++p) {
        if (!H[p].src.empty())
            HIPCHK(hipMemcpy(base + off[p][0], H[p].src.data(), H[p].src.size() * sizeof(int2), hipMemcpyHostToDevice));
        if (!H[p].tgt.empty())
            HIPCHK(hipMemcpy(base + off[p][1], H[p].tgt.data(), H[p].tgt.size() * sizeof(int2), hipMemcpyHostToDevice));
        if (!H[p].coef.empty()) {
            if (f64) {
                HIPCHK(hipMemcpy(base + off[p][2], H[p].coef.data(), H[p].coef.size() * es, hipMemcpyHostToDevice));
            } else {
                std::vector<float> c32(H[p].coef.begin(), H[p].coef.end());
                HIPCHK(hipMemcpy(base + off[p][2], c32.data(), c32.size() * es, hipMemcpyHostToDevice));
            }
        }
        win[p].src = (const int2*)(base + off[p][0]);
        win[p].tgt = (const int2*)(base + off[p][1]);
        win[p].coef = base + off[p][2];
    }
    return PM_OK;
}

// Streams of the forward or transposed tile sweep (layout documented in
// kernels.h), one depth per parity; the couplings are counted as for the window streams.
int build_tile_tables(bool adj, pm::TileArgs (&tile)[2], void** mem) {
    const pm::Layout& L = C.L;
    const int N = C.N, V = C.V, MU1 = N + 2;
    const FluxRows flux(N);
    const long long* nnz_par = flux.nnz_par;
    auto exists = [&](int l, int mu, int ty) { return l >= 0 && l <= N && mu >= 0 && mu <= l && !(ty == 1 && mu == 0); };
    auto idx = [](int l, int mu, int ty) { return l * l + l + (ty == 0 ? mu : -mu); };
    std::vector<uint32_t> src[2], tgt[2];
    const long long unit = C.g.pstride / 64;  // entries count 64 elements
    std::vector<double> coef[2];
    for (int p = 0; p < 2; ++p) {
        const int nd = N >= p ? (N - p) / 2 + 1 : 0;
        const int K = pm::tile_depth(C.prec, nd, adj), npass = (nd + K - 1) / K;
        tile[p] = pm::TileArgs{N, p, K, npass, nullptr, nullptr, nullptr};
        src[p].assign((size_t)npass * MU1 * 2 * (K + 1), 0);
        tgt[p].assign((size_t)npass * MU1 * 2 * K, 0);
        coef[p].assign((size_t)npass * MU1 * 2 * (K + 1) * 10, 0.0);
        long long used = 0;
        for (int pass = 0; pass < npass; ++pass) {
            const int L0 = p + 2 * K * pass;
            for (int mu = 0; mu < MU1; ++mu)
                for (int ty = 0; ty < 2; ++ty) {
                    const size_t col = ((size_t)pass * MU1 + mu) * 2 + ty;
                    for (int t = 0; t < K; ++t)
                        if (exists(L0 + 2 * t, mu, ty))
                            tgt[p][col * K + t] = (uint32_t)((L.slot_of[idx(L0 + 2 * t, mu, ty)] - (p ? (int)C.ve : 0)) * unit);
                    for (int b = 0; b <= K; ++b) {
                        const int ls = L0 - 1 + 2 * b;
                        if (!exists(ls, mu, ty)) continue;
                        const int j = idx(ls, mu, ty);
                        const int bits = pm::grid_bits(ls, ty == 0 ? mu : -mu);
                        src[p][col * (K + 1) + b] = (uint32_t)((L.slot_of[j] - (p ? 0 : (int)C.ve)) * unit);
                        for (int side = 0; side < 2; ++side) {
                            const int t = side == 0 ? b : b - 1;
                            if (t < 0 || t >= K) continue;
                            const int tmu[5] = {mu - 1, mu - 1, mu, mu + 1, mu + 1};
                            const int tty[5] = {ty, 1 - ty, ty, ty, 1 - ty};
                            const int dir[5] = {0, 1, 2, 0, 1};
                            for (int r = 0; r < 5; ++r) {
                                if (!exists(L0 + 2 * t, tmu[r], tty[r])) continue;
                                const double* val = flux.find(idx(L0 + 2 * t, tmu[r], tty[r]), j, dir[r]);
                                if (!val) continue;
                                const double sgn = ((bits >> dir[r]) & 1) ? -1.0 : 1.0;
                                coef[p][((col * (K + 1) + b) * 2 + side) * 5 + r] = sgn * *val / C.h[dir[r]];
                                ++used;
                            }
                        }
                    }
                }
        }
        if (used != nnz_par[p])
            return fail(PM_EINVAL, "internal: tile streams cover " + std::to_string(used) + " of " +
                                       std::to_string(nnz_par[p]) + " couplings");
        const long long nhalf[2] = {C.ve, (long long)V - C.ve};
        for (uint32_t e : src[p])
            if (e >= nhalf[1 - p] * unit) return fail(PM_EINVAL, "internal: source slot outside its half");
        for (uint32_t e : tgt[p])
            if (e >= nhalf[p] * unit) return fail(PM_EINVAL, "internal: target slot outside its half");
    }
    const bool f64 = C.prec == PM_FP64;
    const size_t es = f64 ? sizeof(double) : sizeof(float);
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    std::vector<char> host;
    size_t off[2][3];
    auto put = [&](const void* p, size_t bytes) {
        const size_t at = host.size();
        host.resize(at + up(bytes));
        if (bytes) std::memcpy(host.data() + at, p, bytes);
        return at;
    };
    for (int p = 0; p < 2; ++p) {
        off[p][0] = put(src[p].data(), src[p].size() * sizeof(int));
        off[p][1] = put(tgt[p].data(), tgt[p].size() * sizeof(int));
        std::vector<float> c32(coef[p].begin(), coef[p].end());
        off[p][2] = f64 ? put(coef[p].data(), coef[p].size() * es) : put(c32.data(), c32.size() * es);
    }
    int rc = dmalloc(mem, host.size(), "tile streams");
    if (rc) return rc;
    HIPCHK(hipMemcpy(*mem, host.data(), host.size(), hipMemcpyHostToDevice));
    for (int p = 0; p < 2; ++p) {
        char* base = (char*)*mem;
        tile[p].src = (const uint32_t*)(base + off[p][0]);
        tile[p].tgt = (const uint32_t*)(base + off[p][1]);
        tile[p].coef = base + off[p][2];
    }
    return PM_OK;
}

// Planes and couplings of the low-order sweep (kernels.h).
int build_low_tables() {
    const int N = C.N;
    const FluxRows flux(N);
    std::vector<double> coef[2];
    const long long unit = C.g.pstride / 64;
    auto exists = [&](int l, int mu, int ty) { return l >= 0 && l <= N && mu >= 0 && mu <= l && !(ty == 1 && mu == 0); };
    auto idx = [](int l, int mu, int ty) { return l * l + l + (ty == 0 ? mu : -mu); };
    for (int p = 0; p < 2; ++p) {  // parity of the targets
        long long used = 0;
        for (int l = 0; l <= N; ++l)
            for (int k = 0; k < 2 * l + 1; ++k) {
                const int mu = (k + 1) / 2, ty = k == 0 ? 0 : (k + 1) % 2, at = l * (l - 1) / 2 + k;
                const int j = idx(l, mu, ty), par = l & 1;
                const uint32_t plane = (uint32_t)((C.L.slot_of[j] - (par ? (int)C.ve : 0)) * unit);
                if (par == p) {
                    C.lowa[p].tgt[at] = plane;
                    continue;
                }
                C.lowa[p].src[at] = plane;
                coef[p].resize((size_t)(at + 1) * 10, 0.0);
                const int bits = pm::grid_bits(l, ty == 0 ? mu : -mu);
                for (int side = 0; side < 2; ++side)
                    for (int r = 0; r < 5; ++r) {
                        const int lt = side == 0 ? l + 1 : l - 1, tmu = r < 2 ? mu - 1 : r == 2 ? mu : mu + 1;
                        const int tty = r == 1 || r == 4 ? 1 - ty : ty, dir = r == 2 ? 2 : r == 1 || r == 4 ? 1 : 0;
                        const double* val = exists(lt, tmu, tty) ? flux.find(idx(lt, tmu, tty), j, dir) : nullptr;
                        if (!val) continue;
                        coef[p][((size_t)at * 2 + side) * 5 + r] = (((bits >> dir) & 1) ? -1.0 : 1.0) * *val / C.h[dir];
                        ++used;
                    }
            }
        if (used != flux.nnz_par[p])
            return fail(PM_EINVAL, "internal: low-order couplings cover " + std::to_string(used) + " of " +
                                       std::to_string(flux.nnz_par[p]));
    }
    const size_t es = C.prec == PM_FP64 ? sizeof(double) : sizeof(float), half = pm::kLowPlanes * 10 * sizeof(double);
    int rc = dmalloc(&C.low_mem, 2 * half, "low-order couplings");
    if (rc) return rc;
    for (int p = 0; p < 2; ++p) {
        const std::vector<float> c32(coef[p].begin(), coef[p].end());
        const void* from = C.prec == PM_FP64 ? (const void*)coef[p].data() : (const void*)c32.data();
        HIPCHK(hipMemcpy((char*)C.low_mem + p * half, from, coef[p].size() * es, hipMemcpyHostToDevice));
        C.lowa[p].coef = (char*)C.low_mem + p * half;
    }
    return PM_OK;
}

// A forward sweep of a state in `base` on the path of the context.
hipError_t forward(void* base, int parity, const pm::StateOffs& so, int rowbase, double tau) {
    if (C.low)
        return pm::launch_sweep_low(C.prec, C.N, parity, base, so, C.tab, C.tabf, rowbase, C.lowa[parity], C.g, C.stream());
    if (C.tiled)
        return pm::launch_sweep_tile(C.prec, base, so, C.tab, C.tabf, rowbase, C.tile[parity], C.tg, C.g, C.stream());
    const pm::Aniso an{C.aniso ? C.gl : nullptr, tau, 0};
    return pm::launch_sweep_win(C.prec, base, so, C.tab, C.tabf, rowbase, an, C.win[parity], C.g, C.stream());
}

// One sweep of the given parity; `full` selects tau = dt for the odd grids
// (two merged odd half steps).
int sweep(void* u, int parity, bool full = false) {
    if (C.passes(parity) == 0) return PM_OK;
    hipEvent_t a = nullptr, b = nullptr;
    if (C.timing) {
        HIPCHK(hipEventCreate(&a));
        HIPCHK(hipEventCreate(&b));
        HIPCHK(hipEventRecord(a, C.stream()));
    }
    const double tau = parity == 0 || full ? C.dt : 0.5 * C.dt;
    const int rowbase = parity == 0 ? 0 : full && !C.aniso ? pm::kTabOddFull : 8;
    const pm::StateOffs so{C.half(1 - parity), C.half(parity), C.half(parity), 0, 0};
    HIPCHK(forward(u, parity, so, rowbase, tau));
    if (C.timing) {
        HIPCHK(hipEventRecord(b, C.stream()));
        C.ev[parity].push_back({a, b});
    }
    return PM_OK;
}

int full_step(void* u) {
    int rc;
    if ((rc = sweep(u, 1))) return rc;
    if ((rc = sweep(u, 0))) return rc;
    return sweep(u, 1);
}

// n steps of eq. (6).  With merging, the trailing odd half step of a step
// and the leading one of the next see the same (unchanged) even moments and
// the odd moments carry no source, so together they are one odd substep of
// length dt (alpha_h^2 = alpha_dt, beta_h (1 + alpha_h) = beta_dt): n steps
// take 2n + 1 sweeps instead of 3n.  The result differs by rounding only.
int run_steps(void* u, long long n, bool merged) {
    if (n <= 0) return PM_OK;
    if (!merged) {
        for (long long s = 0; s < n; ++s) {
            int rc = full_step(u);
            if (rc) return rc;
        }
        return PM_OK;
    }
    int rc;
    if ((rc = sweep(u, 1))) return rc;
    for (long long s = 0; s < n; ++s) {
        if ((rc = sweep(u, 0))) return rc;
        if ((rc = sweep(u, 1, s + 1 < n))) return rc;
    }
    return PM_OK;
}

// Halo faces of a sweep of parity p when the box is one GPU's share of a
// split grid.  The sweep reads each dual moment (parity 1 - p) at one
// neighbour per direction d: forward (c + e_d) when the moment is
// unstaggered in d, backward when it is staggered.  So the -d neighbour
// needs this box's layer 0 of the dual moments unstaggered in d (face d-)
// and the +d neighbour its last layer of those staggered in d (face d+).
// Packing order: faces x-, x+, y-, y+, z-, z+; in a face the moments by
// storage slot, then the face cells with the two other coordinates in
// memory order.
HaloPlan halo_plan(const pm::Layout& L, int nx, int ny, int nz, int parity) {
    HaloPlan hp;
    const long long n[3] = {nx, ny, nz};
    long long end = 0;
    for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, side = f & 1;
        hp.hf.slot0[f] = (int)hp.slots.size();
        for (int s = 0; s < L.V; ++s) {
            const int i = L.moment_of[s];
            int l, m;
            pm::moment_lm(i, l, m);
            if ((l & 1) != 1 - parity) continue;
            if (((pm::grid_bits(l, m) >> d) & 1) != side) continue;
            hp.slots.push_back(s);
        }
        const long long cnt = (long long)hp.slots.size() - hp.hf.slot0[f];
        hp.hf.area[f] = n[(d + 1) % 3] * n[(d + 2) % 3];
        hp.hf.layer[f] = side ? (int)n[d] - 1 : 0;
        end += cnt * hp.hf.area[f];
        hp.hf.end[f] = end;
    }
    hp.hf.slot0[6] = (int)hp.slots.size();
    return hp;
}

// The faces of the directions in `dirs` (bit d: direction d split across
// GPUs): the others get no cells, and the packed offsets close up.
pm::HaloFaces halo_masked(pm::HaloFaces hf, int dirs) {
    long long end = 0;
    for (int f = 0; f < 6; ++f) {
        const long long cnt = hf.slot0[f + 1] - hf.slot0[f];
        if (!((dirs >> (f >> 1)) & 1)) hf.area[f] = 0;
        end += cnt * hf.area[f];
        hf.end[f] = end;
    }
    return hf;
}

int check_moment(int moment) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (moment < 0 || moment >= C.V)
        return fail(PM_EINVAL, "moment " + std::to_string(moment) + " out of range [0, " +
                                   std::to_string(C.V) + ")");
    return PM_OK;
}

}  // namespace

extern "C" {

int pm_set_precision(int p) {
    if (p != PM_FP64 && p != PM_FP32 && p != PM_BF16)
        return fail(PM_EINVAL, "unknown precision " + std::to_string(p));
    g_pending_prec = p;
    return PM_OK;
}

int pm_set_scattering(const double* g, int count) {
    if (count < 0 || count > PM_N_MAX)
        return fail(PM_EINVAL, "scattering count must be in [0, " + std::to_string(PM_N_MAX) + "]");
    if (count > 0 && !g) return fail(PM_EINVAL, "scattering moments are NULL");
    for (int l = 0; l < count; ++l)
        if (!std::isfinite(g[l]) || g[l] < -1.0 || g[l] > 1.0)
            return fail(PM_EINVAL, "g[" + std::to_string(l) + "] (degree " + std::to_string(l + 1) +
                                       ") is not finite or outside [-1, 1]");
    g_pending_scat.assign(g, g + count);
    return PM_OK;
}

int pm_init(int N, int nx, int ny, int nz, double dx, double dt, const double* sigma_a,
            const double* sigma_s, const double* q) {
    return pm_init_cells(N, nx, ny, nz, dx, dx, dx, dt, sigma_a, sigma_s, q);
}

int pm_init_cells(int N, int nx, int ny, int nz, double dx, double dy, double dz, double dt,
                  const double* sigma_a, const double* sigma_s, const double* q) {
    if (N < 0 || N > PM_N_MAX) return fail(PM_EINVAL, "N must be in [0, 63]");
    if (nx < 1 || ny < 1 || nz < 1) return fail(PM_EINVAL, "grid sizes must be >= 1");
    const long long ncell = (long long)nx * ny * nz;
    if (ncell >= (1LL << 31)) return fail(PM_EINVAL, "more than 2^31 - 1 cells");
    for (double hd : {dx, dy, dz})
        if (!(hd > 0.0) || !std::isfinite(hd))
            return fail(PM_EINVAL, "cell edges dx, dy, dz must be positive and finite");
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(PM_EINVAL, "dt must be positive and finite");
    if (!sigma_a || !sigma_s) return fail(PM_EINVAL, "sigma_a and sigma_s are required");
    std::string msg;
    if (!finite_nonneg(sigma_a, ncell, "sigma_a", msg) || !finite_nonneg(sigma_s, ncell, "sigma_s", msg))
        return fail(PM_EINVAL, msg);
    if (q)
        for (long long i = 0; i < ncell; ++i)
            if (!std::isfinite(q[i])) return fail(PM_EINVAL, "q[" + std::to_string(i) + "] not finite");

    release();
    C.dev = this_device();
    C.N = N;
    C.V = (N + 1) * (N + 1);
    C.nx = nx;
    C.ny = ny;
    C.nz = nz;
    C.ncell = ncell;
    C.h[0] = dx;
    C.h[1] = dy;
    C.h[2] = dz;
    C.dt = dt;
    C.prec = g_pending_prec;
    C.esz = elem_size(C.prec);
    C.g.nx = nx;
    C.g.ny = ny;
    C.g.nz = nz;
    C.g.ncell = ncell;
    C.g.pstride = plane_stride(ncell);
    C.L = pm::make_layout(N);
    C.ve = 0;
    for (int l = 0; l <= N; l += 2) C.ve += 2 * l + 1;
    std::vector<double> gl(N + 1, 0.0);
    gl[0] = 1.0;
    for (int l = 1; l <= N && l - 1 < (int)g_pending_scat.size(); ++l) gl[l] = g_pending_scat[l - 1];
    C.aniso = std::any_of(gl.begin() + 1, gl.end(), [](double v) { return v != 0.0; });
    // sigma = 0 Fourier symbol: stable iff dt * lambda_max * sqrt(sum_d 1/h_d^2) <= 1
    const double lim =
        N > 0 ? 1.0 / (pm::lambda_max(N) * std::sqrt(1.0 / (dx * dx) + 1.0 / (dy * dy) + 1.0 / (dz * dz)))
              : INFINITY;
    C.cfl_warn = dt > lim ? 1 : 0;

    int rc;
    hipError_t e = own_stream(&C.own);
    if (e != hipSuccess) {
        release();
        trim_kept_to_share();
        return fail(PM_EDEVICE, std::string("hipStreamCreate: ") + hipGetErrorString(e));
    }
#define TRY(x)            \
    do {                  \
        rc = (x);         \
        if (rc) {         \
            release();    \
            trim_kept(0); \
            return rc;    \
        }                 \
    } while (0)
    {
        size_t fr = 0;
        hipError_t me = free_memory(&fr);
        const size_t need = C.state_bytes() + sizeof(double) * (pm::kTabRows + 3) * (size_t)ncell +
                            (C.prec != PM_FP64 && !C.aniso ? sizeof(float) * pm::kTabRows * (size_t)ncell : 0);
        if (me != hipSuccess) {
            release();
            trim_kept(0);
            return fail(PM_EDEVICE, std::string("hipMemGetInfo: ") + hipGetErrorString(me));
        }
        if (need > fr) {
            release();
            trim_kept(0);
            return fail(PM_ENOMEM, "context needs " + std::to_string(need) + " bytes, " +
                                       std::to_string(fr) + " free on the device");
        }
    }
    TRY(dmalloc(&C.u, C.state_bytes(), "state"));
    TRY(dmalloc(&C.tab, sizeof(double) * pm::kTabRows * (size_t)ncell, "tables"));
    TRY(dmalloc(&C.sig, sizeof(double) * 2 * (size_t)ncell, "sigma"));
    const bool ftab = C.prec != PM_FP64 && !C.aniso;
    if (ftab) TRY(dmalloc(&C.tabf, sizeof(float) * pm::kTabRows * (size_t)ncell, "float tables"));
    if (C.aniso) TRY(dmalloc(&C.gl, sizeof(double) * gl.size(), "scattering moments"));
    TRY(dmalloc(&C.plane64, sizeof(double) * (size_t)ncell, "plane"));
    TRY(dmalloc(&C.red, sizeof(double) * (std::max(C.npart, C.ncheck) + 1), "reduction"));
    TRY(dmalloc(&C.redc, sizeof(unsigned long long) * (C.ncheck + 1), "reduction"));
    C.low = !C.aniso && pm::low_use(C.prec, N, ncell);
    C.tiled = !C.low && !C.aniso && pm::tile_use(C.prec, N, C.g, C.tg);
    C.low_adj = C.low && N <= pm::kLowAdjMax;
    C.tiled_adj = C.tiled || (C.low && !C.low_adj && C.prec != PM_BF16 && pm::tile_use_adj(C.prec, N, C.g, C.tg));
    const int kwin = pm::win_depth(C.prec, nx, N, C.aniso);
    if (C.low) {
        TRY(build_low_tables());
    } else if (C.tiled) {
        TRY(build_tile_tables(false, C.tile, &C.tile_mem[0]));
    } else {
        TRY(build_window_tables(kwin, C.win, &C.win_mem));
    }
    if (C.tiled_adj) {
        TRY(build_tile_tables(true, C.tadj, &C.tile_mem[1]));
    } else if (C.prec != PM_BF16 && !C.low_adj) {  // transposed window sweeps
        if (C.low || pm::adj_depth(C.prec) != kwin) {
            TRY(build_window_tables(pm::adj_depth(C.prec), C.wadj, &C.adj_mem));
        } else {
            C.wadj[0] = C.win[0];
            C.wadj[1] = C.win[1];
        }
    }
    hipStream_t s = C.stream();
    auto dev = [&](hipError_t err, const char* what) -> int {
        if (err == hipSuccess) return PM_OK;
        return fail(PM_EDEVICE, std::string(what) + ": " + hipGetErrorString(err));
    };
    if (C.low) TRY(dev(pm::low_load(), "loading kernels"));
    if (C.tiled_adj) TRY(dev(pm::tile_load(), "loading kernels"));
    for (int p = 0; p < 2; ++p) {
        C.halo[p] = halo_plan(C.L, nx, ny, nz, p);
        TRY(dmalloc(&C.halo_slots[p], sizeof(int) * std::max<size_t>(1, C.halo[p].slots.size()), "halo faces"));
        if (!C.halo[p].slots.empty())
            TRY(dev(hipMemcpyAsync(C.halo_slots[p], C.halo[p].slots.data(), sizeof(int) * C.halo[p].slots.size(),
                                   hipMemcpyHostToDevice, C.stream()),
                    "copy halo faces"));
    }
    TRY(dev(hipMemcpyAsync(C.sig, sigma_a, sizeof(double) * ncell, hipMemcpyHostToDevice, s), "copy sigma_a"));
    TRY(dev(hipMemcpyAsync(C.sig + ncell, sigma_s, sizeof(double) * ncell, hipMemcpyHostToDevice, s), "copy sigma_s"));
    if (q) TRY(dev(hipMemcpyAsync(C.plane64, q, sizeof(double) * ncell, hipMemcpyHostToDevice, s), "copy q"));
    if (C.aniso)
        TRY(dev(hipMemcpyAsync(C.gl, gl.data(), sizeof(double) * gl.size(), hipMemcpyHostToDevice, s),
                "copy scattering moments"));
    TRY(dev(pm::launch_tables(C.sig, C.sig + ncell, q ? C.plane64 : nullptr, C.tab, C.g, dt, C.aniso, s),
            "tables"));
    if (ftab) TRY(dev(pm::launch_tables_f32(C.tab, C.tabf, ncell, s), "float tables"));
    TRY(dev(pm::launch_fill_zero(C.u, (long long)C.state_bytes(), s), "zero state"));
    TRY(dev(hipStreamSynchronize(s), "sync"));
#undef TRY
    dfree(C.sig);
    C.sig = nullptr;
    C.dev_bytes -= (long long)(sizeof(double) * 2 * (size_t)ncell);
    trim_kept_to_share();
    C.base_bytes = C.dev_bytes;
    C.live = true;
    return PM_OK;
}

int pm_write(int moment, const double* src) {
    int rc = check_moment(moment);
    if (rc) return rc;
    if (!src) return fail(PM_EINVAL, "src is NULL");
    hipStream_t s = C.stream();
    const int slot = C.L.slot_of[moment];
    if (C.prec == PM_FP64) {
        HIPCHK(hipMemcpyAsync(C.plane(C.u, slot), src, sizeof(double) * C.ncell, hipMemcpyHostToDevice, s));
    } else {
        HIPCHK(hipMemcpyAsync(C.plane64, src, sizeof(double) * C.ncell, hipMemcpyHostToDevice, s));
        HIPCHK(pm::launch_from_f64(C.prec, C.plane64, C.plane(C.u, slot), C.ncell, s));
    }
    HIPCHK(hipStreamSynchronize(s));
    drop_recording();
    return PM_OK;
}

int pm_write_dev(int moment, const void* dsrc) {
    int rc = check_moment(moment);
    if (rc) return rc;
    if (!dsrc) return fail(PM_EINVAL, "src is NULL");
    const int slot = C.L.slot_of[moment];
    HIPCHK(pm::launch_from_f64(C.prec, (const double*)dsrc, C.plane(C.u, slot), C.ncell, C.stream()));
    drop_recording();
    return PM_OK;
}

int pm_step(int nsteps) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (nsteps < 0) return fail(PM_EINVAL, "nsteps < 0");
    int rc;
    long long done = 0;
    while (done < nsteps) {
        long long chunk = nsteps - done;
        if (C.ck > 0) {
            if (C.rec_steps % C.ck == 0) {
                size_t fr = 0;
                HIPCHK(free_memory(&fr));
                if (C.state_bytes() > fr) return fail(PM_ENOMEM, "no device memory for a checkpoint");
                void* p = nullptr;
                if ((rc = dmalloc(&p, C.state_bytes(), "checkpoint"))) return rc;
                C.ckpts.push_back(p);
                HIPCHK(hipMemcpyAsync(p, C.u, C.state_bytes(), hipMemcpyDeviceToDevice, C.stream()));
            }
            chunk = std::min<long long>(chunk, C.ck - C.rec_steps % C.ck);  // stop at the next checkpoint
        }
        if ((rc = run_steps(C.u, chunk, g_merge != 0))) return rc;
        done += chunk;
        if (C.ck > 0) C.rec_steps += chunk;
    }
    if (C.ck > 0 && nsteps > 0) ++g_rec_id;
    return PM_OK;
}

int pm_set_merge(int on) {
    if (on != 0 && on != 1) return fail(PM_EINVAL, "pm_set_merge takes 0 or 1");
    g_merge = on;
    return PM_OK;
}

int pm_read(int moment, double* dst) {
    int rc = check_moment(moment);
    if (rc) return rc;
    if (!dst) return fail(PM_EINVAL, "dst is NULL");
    hipStream_t s = C.stream();
    const int slot = C.L.slot_of[moment];
    if (C.prec == PM_FP64) {
        HIPCHK(hipMemcpyAsync(dst, C.plane(C.u, slot), sizeof(double) * C.ncell, hipMemcpyDeviceToHost, s));
    } else {
        HIPCHK(pm::launch_to_f64(C.prec, C.plane(C.u, slot), C.plane64, C.ncell, s));
        HIPCHK(hipMemcpyAsync(dst, C.plane64, sizeof(double) * C.ncell, hipMemcpyDeviceToHost, s));
    }
    HIPCHK(hipStreamSynchronize(s));
    return PM_OK;
}

int pm_read_dev(int moment, void* ddst) {
    int rc = check_moment(moment);
    if (rc) return rc;
    if (!ddst) return fail(PM_EINVAL, "dst is NULL");
    const int slot = C.L.slot_of[moment];
    HIPCHK(pm::launch_to_f64(C.prec, C.plane(C.u, slot), (double*)ddst, C.ncell, C.stream()));
    return PM_OK;
}

int pm_set_checkpoint(int k) {
    if (k < 0) return fail(PM_EINVAL, "checkpoint interval < 0");
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (k > 0 && C.prec == PM_BF16)
        return fail(PM_EINVAL, "gradients are not supported for bfloat16 storage");
    drop_recording();
    C.ck = k;
    return PM_OK;
}

// Reverse pass.  The steps run as the merged schedule: the substeps of a run
// of T steps are O(half) E O E ... O E O(half), every inner O a full odd
// substep, and the last half step has no cotangent.  Segments between
// checkpoints are recomputed, last first: from (E_0, O_0) of a checkpoint
// the odd states P = O'_0 (after its opening half step), O'_1 .. O'_{len-1}
// and the even states E_1 .. E_len, a substep writing its own half into a
// fresh buffer.  The transposed substeps (launch_adj_*) need the target's
// values before and after: (E_j, E_{j+1}) for an even one, (O'_{j-1}, O'_j)
// for an odd one; the odd substep between two segments runs from the earlier
// one's last O' to the later one's P, kept in a buffer of its own.
}  // extern "C"

namespace {

// Reverse pass; dL_du0, dsa and dss are host pointers (dev = false) or
// device pointers (dev = true).
int grad_impl(const double* dL_du0, double* dsa, double* dss, bool dev) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (C.ck <= 0) return fail(PM_ESTATE, "no gradient recording: call pm_set_checkpoint(k > 0) before pm_step");
    if (!dL_du0) return fail(PM_EINVAL, "dL_du0 is NULL");
    hipStream_t s = C.stream();
    const long long n = C.ncell;
    const long long T = C.rec_steps;
    const int ck = C.ck;
    const long long ps = C.g.pstride;
    const long long SE = (long long)C.V * ps;      // elements of a state
    const long long EH = C.ve * ps;                 // elements of the even half
    const long long OH = SE - EH;                   // elements of the odd half
    const int segs = T > 0 ? (int)std::min<long long>(ck, T) : 1;
    const long long pool_elems = SE + 2 * OH + segs * EH + (segs - 1) * OH;
    void* pool = nullptr;
    double *grad = nullptr, *outg = nullptr, *gpass = nullptr;
    const long long before = C.dev_bytes;
    const bool timing = C.timing;
    auto cleanup = [&]() {
        (void)hipStreamSynchronize(s);
        dfree(pool); dfree(grad); dfree(outg); dfree(gpass);
        trim_kept_to_share();
        C.dev_bytes = before;
        C.timing = timing;
    };
    int rc;
#define TRYG(x)           \
    do {                  \
        rc = (x);         \
        if (rc) {         \
            cleanup();    \
            return rc;    \
        }                 \
    } while (0)
#define HIPG(x)                                                                        \
    do {                                                                               \
        hipError_t e_ = (x);                                                           \
        if (e_ != hipSuccess) {                                                        \
            cleanup();                                                                 \
            return fail(PM_EDEVICE, std::string(#x) + ": " + hipGetErrorString(e_));   \
        }                                                                              \
    } while (0)
    const int np0 = C.adj_passes(0), np1 = C.adj_passes(1);
    const int rows = pm::grad_rows(C.aniso);
    const size_t gpb = sizeof(double) * rows * (size_t)n;  // one pass of gradient rows
    const size_t pool_bytes = C.esz * (size_t)pool_elems;
    {
        size_t fr = 0;
        HIPCHK(free_memory(&fr));
        const size_t need = pool_bytes + gpb * (size_t)(np0 + np1 + 1) + sizeof(double) * 2 * (size_t)n;
        if (need > fr)
            return fail(PM_ENOMEM, "gradient pass needs " + std::to_string(need) + " bytes, " +
                                       std::to_string(fr) + " free on the device");
    }
    TRYG(dmalloc(&pool, pool_bytes, "adjoint and segment states"));
    TRYG(dmalloc(&gpass, gpb * (size_t)(np0 + np1), "per-pass gradient rows"));
    TRYG(dmalloc(&grad, gpb, "gradient accumulators"));
    TRYG(dmalloc(&outg, sizeof(double) * 2 * (size_t)n, "gradient output"));
    // pool layout (elements): w [0, SE), P of even and odd segments, E_1 ..
    // E_len, O'_1 .. O'_{len-1}; the checkpoints are read where they are
    const long long W = 0, P0 = SE, EB = SE + 2 * OH, OB = EB + segs * EH;
    HIPG(pm::launch_fill_zero(pool, (long long)(C.esz * (size_t)SE), s));
    HIPG(pm::launch_fill_zero(gpass, (long long)(gpb * (np0 + np1)), s));
    if (!dev) HIPG(hipMemcpyAsync(C.plane64, dL_du0, sizeof(double) * n, hipMemcpyHostToDevice, s));
    double* gp_par[2] = {gpass, gpass + (size_t)np0 * rows * (size_t)n};
    C.timing = false;
    auto odd_tau = [&](bool full) { return full ? C.dt : 0.5 * C.dt; };
    auto odd_row = [&](bool full) { return full && !C.aniso ? pm::kTabOddFull : 8; };
    auto fwd = [&](int p, long long src, long long tin, long long tout, bool full) -> hipError_t {
        if (C.passes(p) == 0) return hipSuccess;  // a parity without moments (N = 0, odd)
        return forward(pool, p, pm::StateOffs{src, tin, tout, 0, 0}, p ? odd_row(full) : 0, p ? odd_tau(full) : C.dt);
    };
    // transpose of a substep of parity p with the target values pre and post
    auto adj = [&](int p, long long pre, long long post, bool full) -> hipError_t {
        if ((p ? np1 : np0) == 0) return hipSuccess;
        const long long we = W, wo = W + EH;
        const pm::StateOffs so{p ? we : wo, p ? wo : we, p ? wo : we, pre, post};
        const int row = p ? odd_row(full) : 0, opening = p && !full;
        const double tau = p ? odd_tau(full) : C.dt;
        if (C.low_adj)
            return pm::launch_adj_low(C.prec, C.N, p, pool, so, gp_par[p], C.tab, row, tau, opening, C.lowa[p], C.g, s);
        if (C.tiled_adj)
            return pm::launch_adj_tile(C.prec, pool, so, gp_par[p], C.tab, row, tau, opening, C.tadj[p], C.tg, C.g, s);
        return pm::launch_adj_win(C.prec, pool, so, gp_par[p], C.tab, row, pm::Aniso{C.aniso ? C.gl : nullptr, tau, opening},
                                  C.wadj[p], C.g, s);
    };
    const long long nseg = (T + ck - 1) / ck;
    for (long long gseg = nseg - 1; gseg >= 0; --gseg) {
        const long long s0 = gseg * ck, len = std::min<long long>(s0 + ck, T) - s0;
        // the checkpoint's place as an offset from the pool: a difference of
        // addresses (two allocations; both on 256 bytes, so whole elements)
        const long long E0 = ((long long)(intptr_t)C.ckpts[gseg] - (long long)(intptr_t)pool) / (long long)C.esz, O0 = E0 + EH;
        auto P = [&](long long g) { return P0 + (g & 1) * OH; };
        auto E = [&](long long j) { return j == 0 ? E0 : EB + (j - 1) * EH; };
        auto O1 = [&](long long j) { return j == 0 ? P(gseg) : OB + (j - 1) * OH; };
        for (long long j = 0; j < len; ++j) {
            HIPG(j == 0 ? fwd(1, E0, O0, O1(0), false) : fwd(1, E(j), O1(j - 1), O1(j), true));
            HIPG(fwd(0, O1(j), E(j), E(j + 1), false));
        }
        const long long m0 = (long long)C.L.slot_of[0] * ps;
        auto at = [&](long long off) { return (char*)pool + (long long)C.esz * off; };
        if (gseg == nseg - 1) {
            HIPG(pm::launch_adj_seed(C.prec, dev ? dL_du0 : C.plane64, at(W + m0), at(E(len - 1) + m0), at(E(len) + m0), C.tab,
                                     C.aniso, C.dt, gp_par[0], n, s));
        } else {
            HIPG(adj(1, O1(len - 1), P(gseg + 1), true));
            HIPG(adj(0, E(len - 1), E(len), false));
        }
        for (long long j = len - 1; j >= 1; --j) {
            HIPG(adj(1, O1(j - 1), O1(j), true));
            HIPG(adj(0, E(j - 1), E(j), false));
        }
        if (gseg == 0) HIPG(adj(1, O0, O1(0), false));  // the opening half step
    }
    HIPG(pm::launch_grad_sum(gpass, np0 + np1, grad, rows * n, s));
    if (dev) {
        HIPG(pm::launch_grad_final(grad, dsa, dss, C.g, C.aniso, s));
    } else {
        HIPG(pm::launch_grad_final(grad, outg, outg + n, C.g, C.aniso, s));
        if (dsa) HIPG(hipMemcpyAsync(dsa, outg, sizeof(double) * n, hipMemcpyDeviceToHost, s));
        if (dss) HIPG(hipMemcpyAsync(dss, outg + n, sizeof(double) * n, hipMemcpyDeviceToHost, s));
    }
    // the temporaries are freed below: the queued work must be done first
    HIPG(hipStreamSynchronize(s));
    cleanup();
#undef TRYG
#undef HIPG
    return PM_OK;
}

}  // namespace

extern "C" {

int pm_grad(const double* dL_du0, double* dsa, double* dss) {
    return grad_impl(dL_du0, dsa, dss, false);
}

int pm_grad_dev(const void* dL_du0, void* dsa, void* dss) {
    return grad_impl((const double*)dL_du0, (double*)dsa, (double*)dss, true);
}

long long pm_recording_id(void) { return g_rec_id; }

int pm_total(double* out) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (!out) return fail(PM_EINVAL, "out is NULL");
    hipStream_t s = C.stream();
    HIPCHK(pm::launch_sum(C.prec, C.plane(C.u, C.L.slot_of[0]), C.ncell, C.red, C.npart,
                          C.red + C.npart, s));
    HIPCHK(hipMemcpyAsync(out, C.red + C.npart, sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return PM_OK;
}

int pm_check(double* max_abs, long long* n_nonfinite) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    hipStream_t s = C.stream();
    HIPCHK(pm::launch_check(C.prec, C.u, C.V, C.g, C.red, C.redc, C.ncheck, C.red + C.ncheck,
                            C.redc + C.ncheck, s));
    double m = 0;
    unsigned long long k = 0;
    HIPCHK(hipMemcpyAsync(&m, C.red + C.ncheck, sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(hipMemcpyAsync(&k, C.redc + C.ncheck, sizeof(k), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (max_abs) *max_abs = m;
    if (n_nonfinite) *n_nonfinite = (long long)k;
    if (k) return fail(PM_ENONFINITE, std::to_string(k) + " non-finite values in the state");
    return PM_OK;
}

int pm_check_noalloc(void* dev_max_abs, void* dev_nonfinite) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (!dev_max_abs || !dev_nonfinite) return fail(PM_EINVAL, "output pointers must not be NULL");
    const int npart = C.ncheck;
    if (npart > pm::scratch_partials())
        return fail(PM_EINVAL, "pm_check_noalloc: " + std::to_string(npart) + " partial results exceed the " +
                                   std::to_string(pm::scratch_partials()) + " of the static scratch");
    // the scratch's device address: looked up on the first call on a device
    // (hipGetSymbolAddress, return code checked), kept per device
    void* scr = nullptr;
    HIPCHK(pm::scratch_device(&scr));
    double* pmax = (double*)scr;
    unsigned long long* pcnt = (unsigned long long*)((char*)scr + sizeof(double) * pm::scratch_partials());
    // every partial is written before it is read: nothing to clear
    HIPCHK(pm::launch_check(C.prec, C.u, C.V, C.g, pmax, pcnt, npart, (double*)dev_max_abs,
                            (unsigned long long*)dev_nonfinite, C.stream()));
    return PM_OK;
}

int pm_bind_stream(void* stream) {
    g_bound = (hipStream_t)stream;
    return PM_OK;
}

int pm_sync(void) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    HIPCHK(hipStreamSynchronize(C.stream()));
    return PM_OK;
}

int pm_cfl_warning(void) { return C.live ? C.cfl_warn : 0; }

int pm_timing(int on) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    HIPCHK(hipStreamSynchronize(C.stream()));
    drop_events();
    C.timing = on != 0;
    return PM_OK;
}

int pm_sweep_times(int* n_odd, double* ms_odd, int* n_even, double* ms_even) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    HIPCHK(hipStreamSynchronize(C.stream()));
    double t[2] = {0, 0};
    for (int p = 0; p < 2; ++p)
        for (auto& pr : C.ev[p]) {
            float ms = 0;
            HIPCHK(hipEventElapsedTime(&ms, pr.first, pr.second));
            t[p] += ms;
        }
    if (n_odd) *n_odd = (int)C.ev[1].size();
    if (ms_odd) *ms_odd = t[1];
    if (n_even) *n_even = (int)C.ev[0].size();
    if (ms_even) *ms_even = t[0];
    return PM_OK;
}

void pm_finalize(void) {
    if (C.live || C.u || C.own) {
        if (C.own || g_bound) (void)hipStreamSynchronize(C.stream());
        release();
    }
    trim_kept(0);
    if (g_own) (void)hipStreamDestroy(g_own);
    g_own = nullptr;
}

const char* pm_last_error(void) { return g_err.c_str(); }

int pm_flux_nnz(int N) {
    if (N < 0 || N > PM_N_MAX) return fail(PM_EINVAL, "N must be in [0, 63]");
    return (int)pm::flux_entries(N).size();
}

int pm_flux_entries(int N, int* row, int* col, int* dir, double* value, int cap) {
    if (N < 0 || N > PM_N_MAX) return fail(PM_EINVAL, "N must be in [0, 63]");
    if (cap < 0) return fail(PM_EINVAL, "cap < 0");
    std::vector<pm::FluxEntry> e = pm::flux_entries(N);
    int k = 0;
    for (; k < (int)e.size() && k < cap; ++k) {
        if (row) row[k] = e[k].row;
        if (col) col[k] = e[k].col;
        if (dir) dir[k] = e[k].dir;
        if (value) value[k] = e[k].val;
    }
    return k;
}

int pm_moment_grid(int N, int moment) {
    if (N < 0 || N > PM_N_MAX) return fail(PM_EINVAL, "N must be in [0, 63]");
    if (moment < 0 || moment >= (N + 1) * (N + 1)) return fail(PM_EINVAL, "moment out of range");
    int l, m;
    pm::moment_lm(moment, l, m);
    return pm::grid_bits(l, m);
}

int pm_moment_slot(int N, int moment) {
    if (N < 0 || N > PM_N_MAX) return fail(PM_EINVAL, "N must be in [0, 63]");
    if (moment < 0 || moment >= (N + 1) * (N + 1)) return fail(PM_EINVAL, "moment out of range");
    return pm::make_layout(N).slot_of[moment];
}

long long pm_halo_plan(int N, int nx, int ny, int nz, int parity, int dirs, long long* moment,
                       long long* cell, long long cap) {
    if (N < 0 || N > PM_N_MAX) return fail(PM_EINVAL, "N must be in [0, 63]");
    if (nx < 1 || ny < 1 || nz < 1) return fail(PM_EINVAL, "grid sizes must be >= 1");
    if (parity != 0 && parity != 1) return fail(PM_EINVAL, "parity must be 0 or 1");
    if (dirs < 1 || dirs > 7) return fail(PM_EINVAL, "dirs must be a nonzero mask of bits 1 (x), 2 (y), 4 (z)");
    if (cap < 0) return fail(PM_EINVAL, "cap < 0");
    const pm::Layout L = pm::make_layout(N);
    HaloPlan hp = halo_plan(L, nx, ny, nz, parity);
    hp.hf = halo_masked(hp.hf, dirs);
    const long long total = hp.hf.end[5];
    if (moment || cell) {
        long long k = 0;
        for (int f = 0; f < 6 && k < cap; ++f) {
            if (hp.hf.area[f] == 0) continue;
            const int d = f >> 1, layer = hp.hf.layer[f];
            const long long cnt = hp.hf.slot0[f + 1] - hp.hf.slot0[f];
            for (long long j = 0; j < cnt && k < cap; ++j)
                for (long long a = 0; a < hp.hf.area[f] && k < cap; ++a, ++k) {
                    long long c;
                    if (d == 0)
                        c = layer + (long long)nx * a;
                    else if (d == 1)
                        c = (a % nx) + (long long)nx * (layer + (long long)ny * (a / nx));
                    else
                        c = a + (long long)nx * ny * layer;
                    if (moment) moment[k] = L.moment_of[hp.slots[hp.hf.slot0[f] + j]];
                    if (cell) cell[k] = c;
                }
        }
    }
    return total;
}

namespace {

int halo_move(int parity, int dirs, void* buf, bool unpack) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (parity != 0 && parity != 1) return fail(PM_EINVAL, "parity must be 0 or 1");
    if (dirs < 1 || dirs > 7) return fail(PM_EINVAL, "dirs must be a nonzero mask of bits 1 (x), 2 (y), 4 (z)");
    if (!buf) return fail(PM_EINVAL, "buffer is NULL");
    const pm::HaloFaces hf = halo_masked(C.halo[parity].hf, dirs);
    HIPCHK(pm::launch_halo(C.prec, unpack, C.u, buf, C.halo_slots[parity], hf, C.g, C.stream()));
    return PM_OK;
}

}  // namespace

int pm_halo_pack(int parity, int dirs, void* device_buf) {
    return halo_move(parity, dirs, device_buf, false);
}

int pm_halo_unpack(int parity, int dirs, const void* device_buf) {
    return halo_move(parity, dirs, const_cast<void*>(device_buf), true);
}

int pm_sweep_kind(int transposed) {
    if (!C.live) return fail(PM_ESTATE, "no context: call pm_init first");
    if (transposed != 0 && transposed != 1) return fail(PM_EINVAL, "pm_sweep_kind takes 0 or 1");
    if (transposed && C.prec == PM_BF16)
        return fail(PM_EINVAL, "gradients are not supported for bfloat16 storage");
    if (transposed ? C.low_adj : C.low) return PM_SWEEP_LOW;
    return (transposed ? C.tiled_adj : C.tiled) ? PM_SWEEP_TILE : PM_SWEEP_WINDOW;
}

long long pm_device_bytes(void) {
    return C.live ? C.base_bytes + (long long)C.ckpts.size() * (long long)C.state_bytes() : 0;
}

}  // extern "C"
