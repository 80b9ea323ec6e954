// lf2_api.cpp -- plans, validation and the C ABI (include/lf2.h).
//
// A plan holds the per-axis twiddle tables (FP64 on the device, rounded once
// to FP32), the integer wavevector tables used by the binning, lazily built
// k^2 tables (per lattice spacing) and shell tables (per bin count).  The
// pass sequence per call:
//   r2c forward : x r2c (in -> out), y (out), z (out)
//   c2r         : z (in -> W), y (W), x c2r (W -> out)       input untouched
//   c2c         : x (in -> out), y (out), z (out) / z, y, x backward
//   Poisson     : x r2c (rho -> W), y (W), z fwd * -1/(N k^2) * z bwd with
//                 optional binning (W), y bwd (W), x c2r (W -> phi)
//   P(k)        : x, y (into W), z forward with a read-only binning epilogue
// followed, when binning, by a fixed-order FP64 reduction and finalize.
#include "../../include/lf2.h"

#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <cmath>
#include <mutex>
#include <string>
#include <vector>

#include "lf2_device.hpp"
#include "lf2_internal.hpp"
#include "lf2_plan.hpp"

using namespace lf2;

namespace lf2 {
namespace host {

thread_local std::string g_err;

lf2_status fail(lf2_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

constexpr int kMaxDevices = 64;

// Shared workspace per device (the paper's temporary memory shared by plans).
struct SharedWs {
    std::mutex mu;
    void *ptr = nullptr;
    size_t bytes = 0;
};
SharedWs g_ws[kMaxDevices];

int64_t gcd64(int64_t a, int64_t b)
{
    while (b) {
        int64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}

// Columns of a run-time-schedule strided tile of lines of L points: as many
// as fit the block's LDS (at most 64), 0 if not even one does.
int gs_cols(const lf2_plan_s *p, int L, int nbins)
{
    int b = 64;
    while (b > 0 && gs_lds_bytes(L, b, nbins) > p->lds_max) --b;
    return b;
}

// Rows of a run-time-schedule x tile: about 4096 complex values per tile (as
// the compiled x tiles), fewer if the LDS does not hold them, 0 if not even
// one row fits.
int gx_rows(const lf2_plan_s *p, int M, int nc)
{
    int rb = 4096 / (M * nc);
    rb = rb < 1 ? 1 : rb > 256 ? 256 : rb;
    while (rb > 0 && gx_lds_bytes(M, nc, rb) > p->lds_max) --rb;
    return rb;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// ------------------------------------------------------------- kernel timing
namespace prof {
struct Rec {
    int id;
    hipEvent_t a, b;
    double bytes;
};
struct Agg {
    int64_t n = 0;
    double ms = 0.0, bytes = 0.0;
};
std::mutex mu;
std::atomic<bool> on{false};
std::vector<std::string> names;
std::vector<Agg> agg;
std::vector<Rec> recs;
std::vector<hipEvent_t> pool;

hipEvent_t take()
{
    if (!pool.empty()) {
        hipEvent_t e = pool.back();
        pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// Set while a call that must not allocate runs on this thread: its launches
// are not recorded (recording may create events).
thread_local bool t_quiet = false;

// Whether launches on this thread are recorded (their names need not be
// made otherwise: about 1 us of a call's host time per pass).
bool active() { return on.load(std::memory_order_relaxed) && !t_quiet; }

// Returns a record index, or -1 when timing is off.
int begin(const std::string &name, double bytes, hipStream_t s)
{
    if (t_quiet) return -1;
    std::lock_guard<std::mutex> lk(mu);
    if (!on) return -1;
    int id = -1;
    for (size_t i = 0; i < names.size(); ++i)
        if (names[i] == name) id = (int)i;
    if (id < 0) {
        names.push_back(name);
        agg.emplace_back();
        id = (int)names.size() - 1;
    }
    Rec r{id, take(), take(), bytes};
    if (!r.a || !r.b) return -1;
    (void)hipEventRecord(r.a, s);
    recs.push_back(r);
    return (int)recs.size() - 1;
}

void end(int idx, hipStream_t s)
{
    if (idx < 0) return;
    std::lock_guard<std::mutex> lk(mu);
    if (idx < (int)recs.size()) (void)hipEventRecord(recs[idx].b, s);
}

void drain()
{
    for (Rec &r : recs) {
        float ms = 0.f;
        if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
            agg[r.id].n += 1;
            agg[r.id].ms += ms;
            agg[r.id].bytes += r.bytes;
        }
        pool.push_back(r.a);
        pool.push_back(r.b);
    }
    recs.clear();
}

void reset()
{
    drain();
    names.clear();
    agg.clear();
}
}  // namespace prof

std::string kname(const char *fmt, ...)
{
    char buf[128];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return buf;
}

lf2_status plan_alloc(lf2_plan p, void **dst, size_t bytes)
{
    void *ptr = nullptr;
    hipError_t e = hipMalloc(&ptr, bytes < 256 ? 256 : bytes);
    if (e != hipSuccess)
        return fail(LF2_ERR_OUT_OF_MEMORY, "hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
    p->allocs.push_back(ptr);
    *dst = ptr;
    return LF2_OK;
}

// Bytes of spectrum-sized workspace W for a call.
size_t spectrum_bytes(const lf2_plan_s *p)
{
    return (size_t)p->nxk * p->n[1] * p->n[2] * p->nc * 8;
}

int x_grid_blocks(const lf2_plan_s *p)
{
    const int rb = p->gen[0] && !p->nat[0] ? p->gen_rb : x_rows_per_block(p->len[0], p->nc);
    return (int)((p->n[1] * p->n[2] + rb - 1) / rb);
}

// Whether the plan's planes run both their axes in one block (k_plane): they
// fit its LDS, the field is small enough to be bound by latency, and the blocks
// fill the chip: planes that take a CU alone (past half its LDS) pay where they
// are three quarters of the CUs' number up to that number, smaller planes of
// that kind (128 KB) from fewer on.  With N1 = 64 and N0 = 64 or 128, real: 4.2 M
// sites 1.2 times faster forward and 1.1 backward, 8.4 M sites equal forward
// and 0.9 times as fast backward.  128 x 128 planes (140 KB), one launch and two
// passes, forward / backward / Poisson solve in us: 128 of them 22.6 / 22.8 / 42.7
// and 23.7 / 22.5 / 41.4, 192 25.5 / 25.2 / 52.2 and 31.4 / 27.7 / 52.5, 240 25.5 /
// 26.1 / 56.9 and 33.4 / 28.1 / 56.7, 256 25.5 / 26.4 / 54.9 and 35.1 / 28.8 / 56.5,
// 270 38.3 / 39.7 / 69.4 and 37.2 / 31.3 / 61.1; 96 x 96 complex planes, 192 of
// them, 27.7 / 26.5 and 31.8 / 28.7; 120 x 120 planes (123 KB), 120 of them: 1.1 and
// 1.03 times faster.
bool plane_fits(const lf2_plan_s *p)
{
    if (p->ntot * p->nc * (p->kind == LF2_C2C ? 2 : 1) > kPlaneFloats) return false;
    if (!plane_axis_ok(p->len[0]) || !plane_axis_ok(p->len[1])) return false;
    const size_t lds = p->lds_max < kPlaneLds ? p->lds_max : kPlaneLds;
    const size_t most = p->n[2] > p->ncu       ? lds / 2
                        : 4 * p->n[2] >= 3 * p->ncu ? lds
                        : lds < 128 * 1024     ? lds
                                               : 128 * 1024;
    return plane_lds_bytes(p->len[0], (int)p->nxk, p->nc, p->len[1]) <= most;
}

// Tile settings of the y and z passes until one is set or tuned.  Narrow tiles
// with normal accesses, except where another setting measured faster (us a pass,
// forward / backward), on spectra past the memory-side cache (256 MB):
//  - y lines of 768 points and more: wide tiles, whose row segments the narrow
//    ones' 64 bytes cut a cache line short (768^3 real 960 / 947 -> 859 / 839,
//    1024^3 real 2140 / 2104 -> 1905 / 1832; 128 x 2048 x 64 complex with three
//    components 206 / 214 -> 182 / 189; 640^3 474 -> 482).  Smaller spectra lose
//    by them: 512 x 1024 x 64 complex (256 MB) 99 / 105 -> 112 / 110, 96 x 1024 x
//    96 complex 35 / 30 -> 41 / 38, 256 x 768 x 128 real 58 / 48 -> 59 / 53;
//  - z lines: wide tiles over 2048 points (256 x 512 x 2048 real 1552 / 1310 ->
//    741 / 688, 256 x 256 x 2048 complex 769 / 971 -> 582 / 592), nontemporal
//    over 1024 points (1024^3 real 2092 / 2115 -> 1942 / 1901, 512 x 512 x 1024
//    complex 1531 / 1675 -> 1043 / 1096), and over 512, 640 and 768 points where
//    the rows' stride is a multiple of 64 KB, so that a tile's rows fall on few
//    memory channels (512^3 complex 596 / 577 -> 434 / 426, 512 x 512 x 640
//    complex 922 / 994 -> 681 / 717, 512 x 384 x 768 complex 620 / 639 -> 566 /
//    600). At other strides 640 and 768 points take them forward alone (768^3
//    real 947 -> 905 and 899 -> 880 on two cards, 640^3 538 -> 504 and 472 ->
//    478; back 875 -> 929, 876 -> 944, 528 -> 531, 491 -> 517, 384 x 512 x 768
//    270 -> 308).  (Register tiles over 1024 and 2048 points are faster still,
//    1845 / 1830 and 887 / 928 of these, but round otherwise: the 1024^3 real
//    pair's error against 64 bits grew from 2.99e-7 to 3.20e-7.  A plan runs them
//    when they are asked for);
//  - the other backward z passes of lines of 320 points and more, which read a
//    spectrum not written just before, from 430 MB on: nontemporal (512^3 real
//    235 -> 215, 384^3 complex 206 -> 178; 384^3 real, 226 MB, 93 -> 101). Not
//    the run-time-schedule lengths, whose tiles lose by it (back, normal and
//    nontemporal: 540^3 356 and 689, 600^3 455 and 549, 900 x 400 x 900 808 and
//    963, 400 x 400 x 480 complex 334 and 378; 450 points 334 and 302).
// Spectra in the paper's order keep narrow tiles along z, which there are rows of
// one plane (backward, nontemporal: 512 x 256 x 320 with three components 229 ->
// 475, 512^3 251 -> 512). Narrow and wide tiles give the same bits forward.
void default_tiles(lf2_plan_s *p)
{
    const size_t bytes = spectrum_bytes(p);
    const int ly = p->len[1], lz = p->len[2];
    if (bytes <= ((size_t)256 << 20)) return;
    if (!p->gen_only[1] && ly >= 768 && s_wide_supported(ly)) p->svar[1] = p->svar_b[1] = 1;
    if (p->klay != 0 || p->gen_only[2]) return;
    const int64_t stride = 8 * p->nxk * p->nc * p->n[1];
    if (lz == 2048) {
        p->svar[2] = p->svar_b[2] = 1;
    } else if (lz == 1024 || ((lz == 512 || lz == 640 || lz == 768) && stride % 65536 == 0)) {
        p->svar[2] = p->svar_b[2] = 3;
    } else if (lz == 640 || lz == 768) {
        p->svar[2] = 3;
    } else if (lz >= 320 && bytes > ((size_t)430 << 20)) {
        p->svar_b[2] = 2;
    }
}

// Workspace layout: [W spectrum][pk partials][sums][sumsq partials][sumsq];
// the results of the two reductions go straight to the caller's arrays, and
// their places stay so that the size a caller planned for does not change.
struct WsLayout {
    size_t w, part, sums, sq, sqt, total;
};

WsLayout ws_layout(const lf2_plan_s *p, bool need_w, int nbins, bool parseval, bool plane = false)
{
    WsLayout l{};
    size_t off = 0;
    l.w = off;
    off += need_w ? align256(spectrum_bytes(p)) : 0;
    l.part = off;
    off += nbins > 0 ? align256((size_t)kPkGrid * (nbins + 1) * 8) : 0;
    l.sums = off;
    off += nbins > 0 ? align256((size_t)(nbins + 1) * 8) : 0;
    l.sq = off;
    const int64_t sq_rows = x_grid_blocks(p);
    off += parseval ? align256((size_t)(plane && p->n[2] > sq_rows ? p->n[2] : sq_rows) * 8) : 0;
    l.sqt = off;
    off += parseval ? 256 : 0;
    l.total = off;
    return l;
}

lf2_status get_workspace(lf2_plan p, size_t need, char **out)
{
    if (need == 0) {
        *out = nullptr;
        return LF2_OK;
    }
    if (p->own_ws) {
        if (p->own_ws_bytes < need)
            return fail(LF2_ERR_INVALID_ARG, "plan workspace of %zu bytes is smaller than the %zu needed",
                        p->own_ws_bytes, need);
        *out = (char *)p->own_ws;
        return LF2_OK;
    }
    SharedWs &ws = g_ws[p->device];
    std::lock_guard<std::mutex> lk(ws.mu);
    if (ws.bytes < need) {
        if (ws.ptr) {
            LF2_HIP(hipDeviceSynchronize());
            LF2_HIP(hipFree(ws.ptr));
            ws.ptr = nullptr;
            ws.bytes = 0;
        }
        void *ptr = nullptr;
        hipError_t e = hipMalloc(&ptr, need);
        if (e != hipSuccess)
            return fail(LF2_ERR_OUT_OF_MEMORY, "workspace hipMalloc(%zu) failed: %s", need,
                        hipGetErrorString(e));
        ws.ptr = ptr;
        ws.bytes = need;
    }
    *out = (char *)ws.ptr;
    return LF2_OK;
}

lf2_status check_device(const lf2_plan_s *p)
{
    int dev = -1;
    LF2_HIP(hipGetDevice(&dev));
    if (dev != p->device)
        return fail(LF2_ERR_INVALID_ARG, "plan was made on device %d but device %d is current",
                    p->device, dev);
    return LF2_OK;
}

ModeTables base_tables(const lf2_plan_s *p)
{
    ModeTables mt{};
    mt.nxk = (int)p->nxk;
    mt.n0 = (int)p->n[0];
    mt.n1 = (int)p->n[1];
    mt.half = p->kind == LF2_R2C ? 1 : 0;
    for (int i = 0; i < 3; ++i) {
        mt.k2[i] = nullptr;
        mt.q[i] = p->q[i];
    }
    mt.thresh = nullptr;
    mt.nbins = 0;
    mt.qmax = (double)p->qmax;
    mt.scale_n = 1.0 / (double)p->ntot;
    // below 2^32 whenever N2 > 1 (it is then at most qmax); unused for N2 = 1
    const int64_t uz = p->lcm / p->n[2];
    mt.qz_unit = (uint32_t)(uz * uz);
    // (lcm / N_i)^2 <= qmax < 2^32 for N_i > 1; m = 0 only along N_i = 1
    const int64_t ux = p->lcm / p->n[0], uy = p->lcm / p->n[1];
    mt.qx_unit = (uint32_t)(ux * ux);
    mt.qy_unit = (uint32_t)(uy * uy);
    mt.k2z_unit = mt.k2x_unit = mt.k2y_unit = 0.0;
    return mt;
}

void set_k2_units(ModeTables &mt, const lf2_plan_s *p, double dx, int discrete)
{
    double u[3] = {0.0, 0.0, 0.0};
    if (!discrete)
        for (int i = 0; i < 3; ++i) {
            const double a = 6.283185307179586476925286766559 / ((double)p->n[i] * dx);
            u[i] = a * a;
        }
    mt.k2x_unit = u[0];
    mt.k2y_unit = u[1];
    mt.k2z_unit = u[2];
}

lf2_status get_k2(lf2_plan p, double dx, int discrete, hipStream_t s, const double *out[3],
                  bool lookup_only)
{
    for (auto &e : p->k2)
        if (e.dx == dx && e.discrete == discrete) {
            for (int i = 0; i < 3; ++i) out[i] = e.tab[i];
            return LF2_OK;
        }
    if (lookup_only)
        return fail(LF2_ERR_NOT_READY,
                    "no k^2 table for dx = %g (%s) on this plan yet: an allocating call with "
                    "these arguments builds it", dx, discrete ? "discrete" : "continuous");
    K2Entry e{dx, discrete, {nullptr, nullptr, nullptr}};
    const int64_t cnt[3] = {p->nxk, p->n[1], p->n[2]};
    for (int i = 0; i < 3; ++i) {
        void *ptr;
        lf2_status st = plan_alloc(p, &ptr, (size_t)cnt[i] * 8);
        if (st) return st;
        e.tab[i] = (double *)ptr;
        LF2_HIP(launch_k2_table(e.tab[i], (int)p->n[i], (int)cnt[i], dx, discrete, s));
    }
    p->k2.push_back(e);
    for (int i = 0; i < 3; ++i) out[i] = e.tab[i];
    return LF2_OK;
}

// Whether one step of m = |n_z| (q_xy + m^2 q_u to q_xy + (m + 1)^2 q_u)
// crosses at most one of the thresholds t_1 .. t_{nbins-1}.  A step from
// q < t_b has m^2 q_u <= q < t_b, so it moves q by (2 m + 1) q_u <
// 2 sqrt(t_b q_u) + q_u; if every gap t_{b+1} - t_b is at least that (plus
// one for the rounding of the square root), no step spans two thresholds.
static bool walk_one_step(const std::vector<int64_t> &t, uint32_t qu)
{
    const int nb = (int)t.size() - 1;
    for (int b = 0; b + 1 <= nb - 1; ++b) {
        const double need = 2.0 * std::sqrt((double)t[b] * (double)qu) + (double)qu + 1.0;
        if ((double)(t[b + 1] - t[b]) < need) return false;
    }
    return true;
}

lf2_status get_shell(lf2_plan p, int nbins, hipStream_t s, ShellEntry *out, bool lookup_only)
{
    for (auto &e : p->shells)
        if (e.nbins == nbins) {
            *out = e;
            return LF2_OK;
        }
    if (lookup_only)
        return fail(LF2_ERR_NOT_READY,
                    "no %d-bin shell table on this plan yet: an allocating call with this bin "
                    "count builds it", nbins);
    ShellEntry e{nbins, nullptr, nullptr, nullptr, 0};
    void *ptr;
    lf2_status st = plan_alloc(p, &ptr, (size_t)(nbins + 1) * 8);
    if (st) return st;
    e.thresh = (int64_t *)ptr;
    if ((st = plan_alloc(p, &ptr, (size_t)nbins * 8))) return st;
    e.count = (double *)ptr;
    if ((st = plan_alloc(p, &ptr, (size_t)nbins * 8))) return st;
    e.sumk = (double *)ptr;
    LF2_HIP(launch_thresholds(e.thresh, nbins, p->qmax, s));
    // shell sums over the lattice (plan-time work, kept with the plan)
    const int grid = 512;
    double *pc = nullptr, *pkk = nullptr;
    LF2_HIP(hipMalloc(&pc, (size_t)grid * nbins * 8));
    hipError_t e2 = hipMalloc(&pkk, (size_t)grid * nbins * 8);
    if (e2 != hipSuccess) {
        (void)hipFree(pc);
        return fail(LF2_ERR_OUT_OF_MEMORY, "hipMalloc failed: %s", hipGetErrorString(e2));
    }
    ModeTables mt = base_tables(p);
    mt.thresh = e.thresh;
    mt.nbins = nbins;
    mt.walk1 = 0;
    hipError_t e3 = launch_shell_partials(mt, (int)p->n[1], (int)p->n[2], 0.0, pc, pkk, grid, s);
    if (e3 == hipSuccess) e3 = launch_reduce_cols(pc, grid, nbins, e.count, s);
    if (e3 == hipSuccess) e3 = launch_reduce_cols(pkk, grid, nbins, e.sumk, s);
    if (e3 == hipSuccess) e3 = hipStreamSynchronize(s);
    (void)hipFree(pc);
    (void)hipFree(pkk);
    if (e3 != hipSuccess) return fail(LF2_ERR_DEVICE, "shell table: %s", hipGetErrorString(e3));
    std::vector<int64_t> th((size_t)nbins + 1);
    LF2_HIP(hipMemcpy(th.data(), e.thresh, th.size() * 8, hipMemcpyDeviceToHost));
    e.walk1 = walk_one_step(th, mt.qz_unit) ? 1 : 0;
    p->shells.push_back(e);
    *out = e;
    return LF2_OK;
}

lf2_status check_ptr(const void *ptr, const char *what, size_t align)
{
    if (!ptr) return fail(LF2_ERR_INVALID_ARG, "%s is NULL", what);
    if (((uintptr_t)ptr) % align)
        return fail(LF2_ERR_INVALID_ARG, "%s is not %zu-byte aligned", what, align);
    return LF2_OK;
}

// ------------------------------------------------------------- pass runners

XArgs x_args(const lf2_plan_s *p, const void *in, void *out, bool in_is_x, bool out_is_x,
             bool real_x)
{
    // x-space arrays carry the halo; k-space arrays do not.  Units are the
    // array's elements: floats for real fields, complex for complex ones.
    XArgs a{};
    a.in = in;
    a.out = out;
    a.nrows = p->n[1] * p->n[2];
    a.n1 = (int)p->n[1];
    const int64_t h = p->halo, nc = p->nc;
    // in-place r2c: real rows padded to the spectrum row's 2 Nh floats
    const int64_t xrow = (p->inplace && p->kind == LF2_R2C) ? 2 * p->nh * nc : (p->n[0] + 2 * h) * nc;
    const int64_t xplane = (p->n[1] + 2 * h) * xrow;
    const int64_t xoff = h * nc + h * xrow + h * xplane;
    // k-space rows: natural [N2][N1][Nk]; the paper's r2c order [N1][N2][Nh]
    const int64_t C1 = p->nxk * nc;
    const int64_t krow = p->klay == 1 ? p->n[2] * C1 : C1, kplane = p->klay == 1 ? C1 : p->n[1] * C1;
    (void)real_x;
    if (in_is_x) {
        a.in_off = xoff;
        a.in_row = xrow;
        a.in_plane = xplane;
    } else {
        a.in_off = 0;
        a.in_row = krow;
        a.in_plane = kplane;
    }
    if (out_is_x) {
        a.out_off = xoff;
        a.out_row = xrow;
        a.out_plane = xplane;
    } else {
        a.out_off = 0;
        a.out_row = krow;
        a.out_plane = kplane;
    }
    a.tw = p->tw[0];
    a.tw_post = p->tw_post;
    a.sumsq = nullptr;
    return a;
}

SArgs s_args(const lf2_plan_s *p, int axis, const void *in, void *out, int epi)
{
    SArgs a{};
    a.in = in;
    a.out = out;
    const int64_t C1 = p->nxk * p->nc;
    if (p->klay == 1) {  // r2c in the paper's order [N1][N2][Nh]
        if (axis == 1) {  // y is the slowest dimension; every (k_x, z) column is contiguous
            a.stride = p->n[2] * C1;
            a.ncols_inner = p->n[2] * C1;
            a.outer = 0;
            a.ncols = p->n[2] * C1;
        } else {  // z jumps a row; columns (k_x, y): column f at (f / C1) N2 C1 + f mod C1
            a.stride = C1;
            a.ncols_inner = C1;
            a.outer = p->n[2] * C1;
            a.ncols = p->n[1] * C1;
        }
    } else if (axis == 1) {
        a.stride = C1;
        a.ncols_inner = C1;
        a.outer = p->n[1] * C1;
        a.ncols = p->n[2] * C1;
    } else {
        a.stride = p->n[1] * C1;
        a.ncols_inner = p->n[1] * C1;
        a.outer = 0;
        a.ncols = p->n[1] * C1;
    }
    a.epi = epi;
    a.tw = p->tw[axis];
    a.mt = base_tables(p);
    a.partial = nullptr;
    return a;
}

// z pass between the natural order and the paper's c2c order
SArgs t_args(const lf2_plan_s *p, const void *in, void *out, int epi)
{
    SArgs a = s_args(p, 2, in, out, epi);
    a.t_n0 = p->n[0];
    a.t_n2 = p->n[2];
    a.t_nc = p->nc;
    return a;
}

lf2_status run_strided(const lf2_plan_s *p, int axis, int sign, const SArgs &a, int grid_cap,
                       hipStream_t s, int *grid_used)
{
    const double sb = (double)spectrum_bytes(p);
    const bool epi = (a.epi & (EPI_PK | EPI_PK_AFTER | EPI_POISSON)) != 0;
    const bool tr = (a.epi & (EPI_TSTORE | EPI_TLOAD)) != 0;
    // run-time schedule: lengths without compiled kernels (or with a schedule
    // set), and plain passes whose tuned schedule beat the compiled kernels
    if (!p->nat[axis] && (p->gen_only[axis] || (p->gen[axis] && !epi))) {
        if (tr)
            return fail(LF2_ERR_UNSUPPORTED, "no transposing pass for line length %d", p->len[axis]);
        const bool pk = (a.epi & (EPI_PK | EPI_PK_AFTER)) != 0;
        const int b = gs_cols(p, p->len[axis], pk ? a.mt.nbins : 0);
        if (b < 1)
            return fail(LF2_ERR_UNSUPPORTED, "line length %d with %d bins does not fit a tile",
                        p->len[axis], pk ? a.mt.nbins : 0);
        int t = -1;
        if (prof::active())
            t = prof::begin(kname("k_gs<%d,%d> %s%s%s %lldx%lldx%lld/%d", sign, epi ? 1 : 0,
                                  axis == 1 ? "y" : "z", (a.epi & EPI_POISSON) ? "+poisson" : "",
                                  pk ? "+pk" : "", (long long)p->n[0], (long long)p->n[1],
                                  (long long)p->n[2], p->nc),
                            (a.epi & EPI_STORE) ? 2 * sb : sb, s);
        hipError_t e = launch_gs(sign, a, p->sched[axis], p->len[axis], b, grid_cap, s, grid_used);
        prof::end(t, s);
        if (e != hipSuccess)
            return fail(LF2_ERR_DEVICE, "strided pass (axis %d, L=%d) launch: %s", axis,
                        p->len[axis], hipGetErrorString(e));
        return LF2_OK;
    }
    const bool freg = epi && sign < 0 && (a.epi & EPI_POISSON) && p->fvar == 1 &&
                      fused_reg_supported(p->len[axis]) &&
                      fused_reg_fits(p->len[axis], (a.epi & (EPI_PK | EPI_PK_AFTER)) ? a.mt.nbins : 0);
    const int variant = tr ? 0 : epi ? (freg ? 8 : 0) : sign < 0 ? p->svar[axis] : p->svar_b[axis];
    const int ntm = ((variant & 2) || epi) ? 1 : 0;  // the fused pass always streams
    int t = -1;
    if (prof::active()) {
        // "<kernel symbol> <pass>": the symbol part matches the profiler's name
        const std::string sym = tr ? kname("k_strided_t<%d,%d>", p->len[axis], sign)
                                : freg ? kname("k_fused_r<%d,%d>", p->len[axis], a.mt.k2z_unit > 0.0 ? 1 : 2)
                                : (variant & 1) ? kname("k_strided_w<%d,%d,%d>", p->len[axis], sign, ntm)
                                : (variant & 4) ? kname("k_strided_r<%d,%d,%d>", p->len[axis], sign, ntm)
                                                : kname("k_strided<%d,%d,%d,%d>", p->len[axis], sign,
                                                        epi ? 1 : 0, ntm);
        t = prof::begin(sym + kname(" %s%s%s %lldx%lldx%lld/%d", axis == 1 ? "y" : "z",
                                    (a.epi & EPI_POISSON) ? "+poisson" : "",
                                    (a.epi & (EPI_PK | EPI_PK_AFTER)) ? "+pk" : "",
                                    (long long)p->n[0], (long long)p->n[1], (long long)p->n[2], p->nc),
                        (a.epi & EPI_STORE) ? 2 * sb : sb, s);
    }
    hipError_t e = launch_strided(p->len[axis], sign, a, grid_cap, s, grid_used, variant,
                                  epi ? 16 : p->schunk[axis]);
    prof::end(t, s);
    if (e != hipSuccess)
        return fail(LF2_ERR_DEVICE, "strided pass (axis %d, L=%d) launch: %s", axis, p->len[axis],
                    hipGetErrorString(e));
    return LF2_OK;
}

lf2_status run_x(const lf2_plan_s *p, int which, int sign, const XArgs &a, hipStream_t s)
{
    hipError_t e;
    const bool gen = p->gen[0] && !p->nat[0];
    int t = -1;
    if (prof::active()) {
        const double rb = (double)p->ntot * p->nc * 4.0;  // real field
        const double sb = (double)spectrum_bytes(p);
        // the same layout test the launchers apply to pick the paired fast kernels
        auto paired = [](const void *q, int64_t off, int64_t row, int64_t plane) {
            return ((uintptr_t)q % 8) == 0 && off % 2 == 0 && row % 2 == 0 && plane % 2 == 0;
        };
        static const char *const kModes[] = {"r2c", "c2r", "c2c"};
        const bool v = which == 0 ? paired(a.in, a.in_off, a.in_row, a.in_plane)
                                  : paired(a.out, a.out_off, a.out_row, a.out_plane);
        std::string sym;
        if (gen)
            sym = kname("k_gx<%s>", kModes[which]);
        else if (which == 2 && p->xx)
            sym = kname("k_x_c2c_s64<%s,%d>", p->xx == 2 ? "dpp" : "bpermute", sign);
        else if (which == 2)
            sym = kname("k_x_c2c_v<%d,%d,%d>", p->len[0], p->nc, sign);
        else if (p->nc == 1 && v)
            sym = kname("k_x_%s_v<%d>", kModes[which], p->len[0]);
        else
            sym = kname("k_x_%s<%d,%d>", kModes[which], p->len[0], p->nc);
        t = prof::begin(sym + kname(" %lldx%lldx%lld/%d", (long long)p->n[0], (long long)p->n[1],
                                    (long long)p->n[2], p->nc),
                        which == 2 ? 2 * sb : rb + sb, s);
    }
    if (gen)
        e = launch_gx(which == 0 ? 1 : which == 1 ? 2 : 0, sign, a, p->sched[0], p->len[0], p->nc,
                      p->gen_rb, s);
    else if (which == 0)
        e = launch_x_r2c(p->len[0], p->nc, a, s);
    else if (which == 1)
        e = launch_x_c2r(p->len[0], p->nc, a, s);
    else if (p->xx)
        e = launch_x_c2c_shfl(sign, p->xx == 2, a, s);
    else
        e = launch_x_c2c(p->len[0], p->nc, sign, a, s);
    prof::end(t, s);
    if (e != hipSuccess)
        return fail(LF2_ERR_DEVICE, "x pass (L=%d) launch: %s", p->len[0], hipGetErrorString(e));
    return LF2_OK;
}

// The x and y passes of every plane in one launch: which as for run_x (0 r2c
// forward, 1 c2r backward, 2 c2c).
lf2_status run_plane(const lf2_plan_s *p, int which, int sign, const XArgs &a, hipStream_t s)
{
    int t = -1;
    if (prof::active()) {
        static const char *const kModes[] = {"r2c", "c2r", "c2c"};
        const double rb = (double)p->ntot * p->nc * 4.0, sb = (double)spectrum_bytes(p);
        t = prof::begin(kname("k_plane<%s,%d> xy %lldx%lldx%lld/%d", kModes[which], sign,
                              (long long)p->n[0], (long long)p->n[1], (long long)p->n[2], p->nc),
                        which == 2 ? 2 * sb : rb + sb, s);
    }
    const hipError_t e = launch_plane(which == 0 ? 1 : which == 1 ? 2 : 0, sign, a, p->len[0],
                                      (int)p->nxk, p->nc, (int)p->n[1], (int)p->n[2], p->tw[1], s);
    prof::end(t, s);
    if (e != hipSuccess)
        return fail(LF2_ERR_DEVICE, "plane pass (%dx%d) launch: %s", p->len[0], p->len[1],
                    hipGetErrorString(e));
    return LF2_OK;
}

// The x pass (x) and the y pass in place on its output, forward; or the y
// pass in place on x's input (W) and the x pass, backward.
lf2_status run_xy(const lf2_plan_s *p, int which, int sign, const XArgs &x, void *spec, hipStream_t s,
                  bool plane)
{
    if (plane) return run_plane(p, which, sign, x, s);
    lf2_status st;
    const SArgs y = s_args(p, 1, spec, spec, EPI_STORE);
    if (sign < 0) {
        if ((st = run_x(p, which, sign, x, s))) return st;
        return run_strided(p, 1, sign, y, kStridedGridCap, s, nullptr);
    }
    if ((st = run_strided(p, 1, sign, y, kStridedGridCap, s, nullptr))) return st;
    return run_x(p, which, sign, x, s);
}

// Binning tail: reduce the partials into the caller's arrays.  sq_part
// (with d_parseval): sq_rows per-block sums of squares of the real field.
lf2_status pk_tail(lf2_plan p, const ShellEntry &sh, const double *part, int grid, double dx,
                   double vscale, double *d_pk, double *d_kmean, double *d_count,
                   double *d_parseval, const double *sq_part, int64_t sq_rows, hipStream_t s)
{
    PkTail a{};
    a.partial = part;
    a.rows = grid;
    a.nbins = sh.nbins;
    a.count = sh.count;
    a.sumk = sh.sumk;
    a.norm = dx * dx * dx / (double)p->ntot;
    a.vscale = vscale;
    a.kscale = 6.283185307179586476925286766559 / ((double)p->lcm * dx);
    a.inv_n = 1.0 / (double)p->ntot;
    a.pk = d_pk;
    a.kmean = d_kmean;
    a.count_out = d_count;
    a.parseval = d_parseval;
    a.sq_part = sq_part;
    a.sq_rows = sq_rows;
    LF2_HIP(launch_pk_tail(a, s));
    return LF2_OK;
}

lf2_status check_bins(const lf2_plan_s *p, int32_t nbins)
{
    if (nbins < 0) return fail(LF2_ERR_INVALID_ARG, "nbins %d < 0", nbins);
    if (nbins > kMaxBins) return fail(LF2_ERR_UNSUPPORTED, "nbins %d > %d", nbins, kMaxBins);
    if (nbins > 0) {
        // nbins^2 * qmax must fit the exact integer bin rule
        long double lim = (long double)nbins * nbins * (long double)p->qmax;
        if (lim > 4.0e18L) return fail(LF2_ERR_UNSUPPORTED, "nbins^2 * qmax overflows the integer bin rule");
    }
    return LF2_OK;
}

}  // namespace host
}  // namespace lf2

using namespace lf2::host;

// ===================================================================== C ABI

extern "C" {

const char *lf2_status_string(lf2_status s)
{
    switch (s) {
    case LF2_OK: return "LF2_OK";
    case LF2_ERR_INVALID_ARG: return "LF2_ERR_INVALID_ARG";
    case LF2_ERR_UNSUPPORTED: return "LF2_ERR_UNSUPPORTED";
    case LF2_ERR_OUT_OF_MEMORY: return "LF2_ERR_OUT_OF_MEMORY";
    case LF2_ERR_DEVICE: return "LF2_ERR_DEVICE";
    case LF2_ERR_BUDGET: return "LF2_ERR_BUDGET";
    case LF2_ERR_BUSY: return "LF2_ERR_BUSY";
    case LF2_ERR_NOT_READY: return "LF2_ERR_NOT_READY";
    }
    return "LF2_ERR_UNKNOWN";
}

const char *lf2_last_error(void) { return g_err.c_str(); }

lf2_status lf2_profile_enable(int32_t on)
{
    std::lock_guard<std::mutex> lk(prof::mu);
    prof::reset();
    prof::on = on != 0;
    return LF2_OK;
}

lf2_status lf2_profile_reset(void)
{
    std::lock_guard<std::mutex> lk(prof::mu);
    prof::reset();
    return LF2_OK;
}

int32_t lf2_profile_count(void)
{
    std::lock_guard<std::mutex> lk(prof::mu);
    prof::drain();
    return (int32_t)prof::names.size();
}

lf2_status lf2_profile_get(int32_t i, char *name, size_t name_len, int64_t *launches, double *ms,
                           double *bytes)
{
    std::lock_guard<std::mutex> lk(prof::mu);
    if (i < 0 || i >= (int32_t)prof::names.size())
        return fail(LF2_ERR_INVALID_ARG, "profile index %d out of range", i);
    if (name && name_len > 0) {
        strncpy(name, prof::names[i].c_str(), name_len - 1);
        name[name_len - 1] = 0;
    }
    if (launches) *launches = prof::agg[i].n;
    if (ms) *ms = prof::agg[i].ms;
    if (bytes) *bytes = prof::agg[i].bytes;
    return LF2_OK;
}

const char *lf2_version(void) { return "lf2 0.1.0 gfx950"; }

}  // extern "C"

namespace {

// Whether the x pass can exchange across lanes: c2c rows of 64 points, one
// component, compiled kernels.
bool x_lane_exchange_ok(const lf2_plan_s *p)
{
    return p->kind == LF2_C2C && p->len[0] == 64 && p->nc == 1 && !p->gen[0] && !p->gen_only[0];
}

// Time the x pass's stage exchange (64-point c2c rows: LDS or across
// lanes), the tile variants and XCD chunk sizes of the y and z passes, and the
// candidate radix schedules of the run-time-schedule kernels (every axis
// without a compiled kernel, and the y and z passes as an alternative to
// the compiled ones), on a scratch spectrum of the plan's shape, and keep the
// fastest.  Each is timed in both directions (after a warm-up; a schedule
// backward only where its forward pass may still win; the compiled tile settings
// of the y and z passes in two sweeps, the second of those near the fastest in a
// direction, each keeping its faster times).  The plan's own default
// (default_tiles with chunk 16, compiled ragged tiles, or the first schedule)
// stays unless another beats it by 3 %; the y and z passes may take another
// variant backward than forward (a 512^3 real z pass backward: nontemporal 208
// us, normal 229; forward 198 and 194).  An axis keeps its winner only if whole
// transforms, forward and back, gain by it: a pass repeated on one array finds
// its rows in the memory-side cache as a transform does not (384^3 complex, the
// backward z pass: normal accesses won by 3 % in the repeats and lost by 12 % in
// the transform).  Last, where the plan runs x and y of its planes in one
// launch, that launch against the two passes so tuned.  Without memory for the
// scratch arrays the defaults stay, or the winners of the repeats.
lf2_status autotune(lf2_plan p)
{
    const size_t bytes = spectrum_bytes(p);
    const int64_t h2 = 2 * p->halo;
    const size_t xbytes = (size_t)((p->n[0] + h2) * (p->n[1] + h2) * (p->n[2] + h2)) * p->nc *
                          (p->kind == LF2_R2C ? 4 : 8);
    // a spectrum, an x-space array (or spectrum), and the workspace's spectrum
    void *w = nullptr, *w2 = nullptr, *w3 = nullptr;
    if (hipMalloc(&w, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return LF2_OK;
    }
    const size_t bytes2 = xbytes > bytes ? xbytes : bytes;
    if (hipMalloc(&w2, bytes2) != hipSuccess) {
        (void)hipGetLastError();
        w2 = nullptr;
    } else if (hipMalloc(&w3, bytes) != hipSuccess) {
        (void)hipGetLastError();
        w3 = nullptr;
    }
    hipStream_t s = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr, e2 = nullptr;
    lf2_status st = LF2_OK;
    auto hip_ok = [&](hipError_t e, const char *what) {
        if (e != hipSuccess && st == LF2_OK) st = fail(LF2_ERR_DEVICE, "autotune %s: %s", what, hipGetErrorString(e));
        return st == LF2_OK;
    };
    // mean microseconds of n launches after a warm-up (-1 on failure)
    auto time_it = [&](auto &&launch, int n = 3) -> double {
        hip_ok(launch(), "launch");
        hip_ok(hipEventRecord(e0, s), "record");
        for (int r = 0; r < n; ++r) hip_ok(launch(), "launch");
        hip_ok(hipEventRecord(e1, s), "record");
        float ms = 0.f;
        if (!hip_ok(hipEventSynchronize(e1), "sync") || !hip_ok(hipEventElapsedTime(&ms, e0, e1), "elapsed"))
            return -1.0;
        return 1e3 * ms / n;
    };
    // the same of n forward, then n backward launch(sign)s into f and b
    auto time_dirs = [&](auto &&launch, int n, double &f, double &b) {
        f = b = -1.0;
        hip_ok(launch(-1), "launch");
        hip_ok(hipEventRecord(e0, s), "record");
        for (int r = 0; r < n; ++r) hip_ok(launch(-1), "launch");
        hip_ok(hipEventRecord(e1, s), "record");
        for (int r = 0; r < n; ++r) hip_ok(launch(1), "launch");
        hip_ok(hipEventRecord(e2, s), "record");
        float ms = 0.f, ms2 = 0.f;
        if (!hip_ok(hipEventSynchronize(e2), "sync") || !hip_ok(hipEventElapsedTime(&ms, e0, e1), "elapsed") ||
            !hip_ok(hipEventElapsedTime(&ms2, e1, e2), "elapsed"))
            return;
        f = 1e3 * ms / n;
        b = 1e3 * ms2 / n;
    };
    // both directions of launch(sign) together (-1 on failure, or where the
    // forward pass alone shows that they are no faster than `best`)
    auto time_both = [&](auto &&launch, double best = -1.0) -> double {
        const double f = time_it([&] { return launch(-1); });
        if (f < 0 || (best >= 0 && 1.6 * f > best)) return -1.0;
        const double b = time_it([&] { return launch(1); });
        return b < 0 ? -1.0 : f + b;
    };
    static const int kChunks[] = {16, 4, 64};  // the default first
    const lf2_plan_s def = *p;
    if (hip_ok(hipStreamCreateWithFlags(&s, hipStreamNonBlocking), "stream") &&
        hip_ok(hipEventCreate(&e0), "event") && hip_ok(hipEventCreate(&e1), "event") &&
        hip_ok(hipEventCreate(&e2), "event") &&
        hip_ok(hipMemsetAsync(w, 0, bytes, s), "memset") &&
        (!w2 || hip_ok(hipMemsetAsync(w2, 0, bytes2, s), "memset"))) {
        // x axis without a compiled kernel: its schedules, on dense rows of w2
        if (p->gen_only[0] && w2) {
            const int64_t c1 = p->nxk * p->nc;
            const int64_t xr = p->n[0] * p->nc;  // floats (r2c) or complex (c2c) per row
            auto args = [&](int sign) {
                XArgs a{};
                a.nrows = p->n[1] * p->n[2];
                a.n1 = (int)p->n[1];
                a.tw = p->tw[0];
                a.tw_post = p->tw_post;
                a.in = sign < 0 ? w2 : w;
                a.out = sign < 0 ? w : w2;
                a.in_row = sign < 0 ? xr : c1;
                a.out_row = sign < 0 ? c1 : xr;
                a.in_plane = a.in_row * p->n[1];
                a.out_plane = a.out_row * p->n[1];
                return a;
            };
            double best = -1.0;
            if (p->nat[0]) {  // the compiled tiles first: the default
                best = p->tune_us[0][0] = time_both([&](int sign) {
                    const XArgs a = args(sign);
                    return p->kind == LF2_C2C ? launch_x_c2c(p->len[0], p->nc, sign, a, s)
                           : sign < 0         ? launch_x_r2c(p->len[0], p->nc, a, s)
                                              : launch_x_c2r(p->len[0], p->nc, a, s);
                });
            }
            for (const GSched &sc : sched_candidates(p->len[0])) {
                if (st != LF2_OK) break;
                const double us = time_both([&](int sign) {
                    const int mode = p->kind == LF2_C2C ? 0 : sign < 0 ? 1 : 2;
                    return launch_gx(mode, sign, args(sign), sc, p->len[0], p->nc, p->gen_rb, s);
                }, best);
                if (p->tune_us[0][0] < 0) p->tune_us[0][0] = us;
                if (us >= 0 && (best < 0 || us < 0.97 * best)) {
                    best = us;
                    p->sched[0] = sc;
                    p->nat[0] = false;
                }
            }
            p->tune_us[0][1] = best;
        }
        // 64-point c2c rows: the stage exchange through LDS or across lanes
        if (x_lane_exchange_ok(p) && w2) {
            XArgs a{};
            a.nrows = p->n[1] * p->n[2];
            a.n1 = (int)p->n[1];
            a.tw = p->tw[0];
            a.in = w;
            a.out = w2;
            a.in_row = a.out_row = p->n[0];
            a.in_plane = a.out_plane = p->n[0] * p->n[1];
            double best = -1.0;
            for (int v = 0; v < 3 && st == LF2_OK; ++v) {
                const double us = time_both([&](int sign) {
                    return v == 0 ? launch_x_c2c(64, 1, sign, a, s)
                                  : launch_x_c2c_shfl(sign, v == 2, a, s);
                });
                if (v == 0) p->tune_us[0][0] = us;
                if (us >= 0 && (best < 0 || us < 0.97 * best)) {
                    best = us;
                    p->xx = v;
                }
            }
            p->tune_us[0][1] = best;
        }
        for (int axis = 1; axis <= 2 && st == LF2_OK; ++axis) {
            const bool wide = !p->gen_only[axis] && s_wide_supported(p->len[axis]);
            const bool reg = !p->gen_only[axis] && s_reg_supported(p->len[axis]);
            const SArgs a = s_args(p, axis, w, w, EPI_STORE);
            double best = -1.0;
            if (!p->gen_only[axis] || p->nat[axis]) {
                // two sweeps over the settings (the second over those that may
                // win), each setting keeping its faster time: a setting timed
                // while the chip's clocks or memory state drift is timed again
                // in the other sweep.
                // Order: the nontemporal settings, then the rest; within 3 % the
                // earlier one stays.  Timed in
                // short bursts, the cached-store settings of long-stride passes
                // come out faster than they run inside a transform (the
                // 3-component 512^3 z pass: plain wide tile 1.35-1.37 ms in the
                // tuner, 1.53-1.67 ms in the transforms; nontemporal wide tile
                // 1.33 ms and 1.40-1.42 ms), so ties go to the streaming ones.
                std::vector<TileTime> t;
                for (int pass = 0; pass < 2; ++pass)
                    for (int v = 0; v < 8; ++v) {
                        if (((v & 2) != 0) != (pass == 0)) continue;
                        if ((v & 1) && !wide) continue;
                        if ((v & 4) && (!reg || (v & 1))) continue;
                        for (int c : kChunks) t.push_back({v, c, -1.0, -1.0});
                    }
                double f0 = -1.0, b0 = -1.0;  // fastest of the first sweep
                for (int sweep = 0; sweep < 2 && st == LF2_OK; ++sweep)
                    for (TileTime &x : t) {
                        const bool dflt = x.chunk == p->schunk[axis] &&
                                          (x.variant == p->svar[axis] || x.variant == p->svar_b[axis]);
                        if (st != LF2_OK) break;
                        if (sweep == 1 && !dflt && x.fwd > 1.06 * f0 && x.bwd > 1.06 * b0) continue;
                        double f, b;
                        time_dirs([&](int sign) {
                            return launch_strided(p->len[axis], sign, a, kStridedGridCap, s, nullptr,
                                                  x.variant, x.chunk);
                        }, 2, f, b);
                        if (f >= 0 && (x.fwd < 0 || f < x.fwd)) x.fwd = f;
                        if (b >= 0 && (x.bwd < 0 || b < x.bwd)) x.bwd = b;
                        if (sweep == 0 && f >= 0 && (f0 < 0 || f < f0)) f0 = f;
                        if (sweep == 0 && b >= 0 && (b0 < 0 || b < b0)) b0 = b;
                    }
                const TileChoice c = choose_tiles(
                    t, TileChoice{p->svar[axis], p->svar_b[axis], p->schunk[axis], -1.0, -1.0});
                p->tune_us[axis][0] = c.us_default;
                best = c.us;
                p->svar[axis] = c.fwd;
                p->svar_b[axis] = c.bwd;
                p->schunk[axis] = c.chunk;
            }
            const int b = gs_cols(p, p->len[axis], 0);
            for (const GSched &sc : sched_candidates(p->len[axis])) {
                if (st != LF2_OK || b < 1) break;
                const double us = time_both([&](int sign) {
                    return launch_gs(sign, a, sc, p->len[axis], b, kStridedGridCap, s, nullptr);
                }, best);
                if (p->tune_us[axis][0] < 0) p->tune_us[axis][0] = us;
                if (us >= 0 && (best < 0 || us < 0.97 * best)) {
                    best = us;
                    p->gen[axis] = true;
                    p->nat[axis] = false;
                    p->sched[axis] = sc;
                }
            }
            p->tune_us[axis][1] = best;
        }
        // the winners in whole transforms (w2 laid out as the plan's x-space array)
        if (w2 && w3 && st == LF2_OK) {
            const lf2_plan_s tuned = *p;
            auto take = [&](int i, const lf2_plan_s &from) {  // axis i's settings
                p->svar[i] = from.svar[i];
                p->svar_b[i] = from.svar_b[i];
                p->schunk[i] = from.schunk[i];
                p->gen[i] = from.gen[i];
                p->nat[i] = from.nat[i];
                p->sched[i] = from.sched[i];
                if (i == 0) p->xx = from.xx;
            };
            const bool real = p->kind == LF2_R2C;
            const int fwd = real ? 0 : 2, bwd = real ? 1 : 2;
            // where lf2_fft_execute keeps the backward intermediate
            void *W = !real && p->klay != 2 && p->halo == 0 ? w2 : w3;
            auto one_pair = [&] {
                lf2_status e = run_xy(p, fwd, -1, x_args(p, w2, w, true, false, real), w, s, p->plane);
                if (!e) e = run_strided(p, 2, -1, s_args(p, 2, w, w, EPI_STORE), kStridedGridCap, s, nullptr);
                if (!e) e = run_strided(p, 2, 1, s_args(p, 2, w, W, EPI_STORE), kStridedGridCap, s, nullptr);
                if (!e) e = run_xy(p, bwd, 1, x_args(p, W, w2, false, true, real), W, s, p->plane);
                return e == LF2_OK ? hipSuccess : hipErrorUnknown;
            };
            auto pair = [&] {
                return time_it(one_pair, bytes < ((size_t)16 << 20) ? 10 : bytes < ((size_t)256 << 20) ? 4
                                                                              : 2);
            };
            const bool was_quiet = prof::t_quiet;
            prof::t_quiet = true;
            p->plane = false;
            bool same[3];
            for (int i = 0; i < 3; ++i)
                same[i] = tuned.svar[i] == def.svar[i] && tuned.svar_b[i] == def.svar_b[i] &&
                          tuned.schunk[i] == def.schunk[i] && tuned.gen[i] == def.gen[i] &&
                          tuned.nat[i] == def.nat[i] && (i > 0 || tuned.xx == def.xx) &&
                          memcmp(&tuned.sched[i], &def.sched[i], sizeof(GSched)) == 0;
            for (int i = 0; i < 3; ++i) take(i, def);
            double best = same[0] && same[1] && same[2] && !def.plane ? -1.0 : pair();
            for (int i = 0; i < 3 && st == LF2_OK; ++i) {
                if (same[i]) continue;
                take(i, tuned);
                const double us = pair();
                if (us >= 0 && us < 0.995 * best) {
                    best = us;
                } else {
                    take(i, def);
                    p->tune_us[i][1] = p->tune_us[i][0];
                }
            }
            if (def.plane && st == LF2_OK) {
                p->plane = true;
                const double one = pair();
                if (one >= 0 && best >= 0 && best < 0.97 * one) p->plane = false;
            }
            prof::t_quiet = was_quiet;
        }
        // reported per pass: the mean of the two directions
        for (auto &us : p->tune_us)
            for (double &v : us)
                if (v > 0) v *= 0.5;
    }
    if (s) (void)hipStreamSynchronize(s);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (e2) (void)hipEventDestroy(e2);
    if (s) (void)hipStreamDestroy(s);
    (void)hipFree(w);
    if (w2) (void)hipFree(w2);
    if (w3) (void)hipFree(w3);
    return st;
}

}  // namespace

extern "C" {

lf2_status lf2_fft_plan(lf2_plan *out, const lf2_lattice *lat, int32_t ncomp, lf2_fft_kind kind,
                        uint32_t flags)
{
    if (!out) return fail(LF2_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!lat) return fail(LF2_ERR_INVALID_ARG, "lattice is NULL");
    if (lat->dim != 3) return fail(LF2_ERR_UNSUPPORTED, "dim %d: only 3-d lattices have an FFT", lat->dim);
    if (lat->halo < 0) return fail(LF2_ERR_INVALID_ARG, "halo %d < 0", lat->halo);
    if (kind != LF2_R2C && kind != LF2_C2C) return fail(LF2_ERR_INVALID_ARG, "bad kind %d", (int)kind);
    if (ncomp < 1) return fail(LF2_ERR_INVALID_ARG, "ncomp %d < 1", ncomp);
    if (flags & ~(LF2_PLAN_AUTOTUNE | LF2_IN_PLACE | LF2_KLAYOUT_PAPER))
        return fail(LF2_ERR_UNSUPPORTED, "plan flags 0x%x not supported", flags);
    if ((flags & LF2_IN_PLACE) && lat->halo != 0)
        return fail(LF2_ERR_UNSUPPORTED, "in-place transforms need halo 0");
    for (int i = 0; i < 3; ++i) {
        if (lat->size[i] < 1) return fail(LF2_ERR_INVALID_ARG, "size[%d] = %lld < 1", i, (long long)lat->size[i]);
        if (lat->size[i] > (1 << 20)) return fail(LF2_ERR_UNSUPPORTED, "size[%d] too large", i);
        if (!gen_factorable(lat->size[i]))
            return fail(LF2_ERR_UNSUPPORTED, "size[%d] = %lld must be 2^a 3^b 5^c", i,
                        (long long)lat->size[i]);
    }
    if (kind == LF2_R2C && lat->size[0] % 2)
        return fail(LF2_ERR_UNSUPPORTED, "r2c needs an even size[0] (got %lld)", (long long)lat->size[0]);
    int lens[3] = {(int)(kind == LF2_R2C ? lat->size[0] / 2 : lat->size[0]), (int)lat->size[1],
                   (int)lat->size[2]};
    bool gen_only[3];
    for (int i = 0; i < 3; ++i) {
        gen_only[i] = i == 0 ? !x_supported(lens[0], ncomp) : !s_supported(lens[i]);
        if (gen_only[i] && lens[i] > kGenMaxLen)
            return fail(LF2_ERR_UNSUPPORTED, "line length %d along dimension %d is longer than %d",
                        lens[i], i, kGenMaxLen);
    }
    if (gen_only[2] && (flags & LF2_KLAYOUT_PAPER) && kind == LF2_C2C)
        return fail(LF2_ERR_UNSUPPORTED, "the c2c paper k-space order needs a compiled z length");

    lf2_plan p = new (std::nothrow) lf2_plan_s();
    if (!p) return fail(LF2_ERR_OUT_OF_MEMORY, "plan allocation");
    hipError_t e = hipGetDevice(&p->device);
    if (e != hipSuccess || p->device < 0 || p->device >= kMaxDevices) {
        delete p;
        return fail(LF2_ERR_DEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    }
    int lds = 0;
    if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, p->device) ==
            hipSuccess &&
        lds > 0)
        p->lds_max = (size_t)lds;
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, p->device) == hipSuccess &&
        ncu > 0)
        p->ncu = ncu;
    // compiled kernels where they exist; run-time radix schedules otherwise
    for (int i = 0; i < 3; ++i) {
        p->gen_only[i] = gen_only[i];
        p->gen[i] = gen_only[i];
        p->nat[i] = gen_only[i] && ragged_supported(lens[i]) &&
                    (i > 0 || ncomp == 1 || ncomp == 2 || ncomp == 3 || ncomp == 6);
        const std::vector<GSched> cand = sched_candidates(lens[i]);
        if (!cand.empty()) p->sched[i] = cand[0];
    }
    // the fused Poisson pass keeps its tile in registers where it can (at 32
    // points the LDS-staged tile is as fast)
    p->fvar = fused_reg_supported(lens[2]) && lens[2] >= 64 ? 1 : 0;
    if (p->gen_only[0] && (p->gen_rb = gx_rows(p, lens[0], ncomp)) < 1) {
        delete p;
        return fail(LF2_ERR_UNSUPPORTED, "x lines of %d points with %d components do not fit a tile",
                    lens[0], ncomp);
    }
    for (int i = 1; i < 3; ++i)
        if (p->gen_only[i] && gs_cols(p, lens[i], 0) < 1) {
            delete p;
            return fail(LF2_ERR_UNSUPPORTED, "strided lines of %d points do not fit a tile", lens[i]);
        }

    p->kind = kind;
    p->nc = ncomp;
    p->halo = lat->halo;
    p->flags = flags;
    p->inplace = (flags & LF2_IN_PLACE) != 0;
    p->klay = (flags & LF2_KLAYOUT_PAPER) ? (kind == LF2_R2C ? 1 : 2) : 0;
    for (int i = 0; i < 3; ++i) {
        p->n[i] = lat->size[i];
        p->len[i] = lens[i];
    }
    p->nh = p->n[0] / 2 + 1;
    p->nxk = kind == LF2_R2C ? p->nh : p->n[0];
    p->ntot = p->n[0] * p->n[1] * p->n[2];
    p->lcm = p->n[0];
    p->lcm = p->lcm / gcd64(p->lcm, p->n[1]) * p->n[1];
    p->lcm = p->lcm / gcd64(p->lcm, p->n[2]) * p->n[2];
    p->qmax = 0;
    for (int i = 0; i < 3; ++i) {
        int64_t a = (p->n[i] / 2) * (p->lcm / p->n[i]);
        p->qmax += a * a;
    }
    default_tiles(p);
    p->plane = plane_fits(p);
    p->plane_bits = p->plane &&
                    plane_axis_bits(p->len[0], kind == LF2_R2C ? PLANE_X_REAL : PLANE_X_COMPLEX) &&
                    plane_axis_bits(p->len[1], PLANE_Y);
    hipStream_t s = nullptr;
    lf2_status st = LF2_OK;
    // the fused binning evaluates the bin rule in 32 x 32 -> 64-bit products
    // (qmax < 7.1e8 for every supported line length)
    if (p->qmax >= ((int64_t)1 << 32))
        st = fail(LF2_ERR_UNSUPPORTED, "lattice too large for the exact bin rule");
    for (int i = 0; i < 3 && st == LF2_OK; ++i) {
        st = plan_alloc(p, &p->tw[i], (size_t)p->len[i] * 8);
        if (st == LF2_OK && launch_twiddles(p->tw[i], p->len[i], s) != hipSuccess)
            st = fail(LF2_ERR_DEVICE, "twiddle kernel launch");
    }
    if (st == LF2_OK && kind == LF2_R2C) {
        st = plan_alloc(p, &p->tw_post, (size_t)p->nh * 8);
        if (st == LF2_OK && launch_twiddles(p->tw_post, -(int)p->n[0], s) != hipSuccess)
            st = fail(LF2_ERR_DEVICE, "twiddle kernel launch");
    }
    const int64_t cnt[3] = {p->nxk, p->n[1], p->n[2]};
    for (int i = 0; i < 3 && st == LF2_OK; ++i) {
        void *ptr = nullptr;
        st = plan_alloc(p, &ptr, (size_t)cnt[i] * 8);
        p->q[i] = (int64_t *)ptr;
        if (st == LF2_OK && launch_q_table(p->q[i], (int)p->n[i], (int)cnt[i], p->lcm / p->n[i], s) != hipSuccess)
            st = fail(LF2_ERR_DEVICE, "q table launch");
    }
    if (st == LF2_OK) {
        e = hipDeviceSynchronize();
        if (e != hipSuccess) st = fail(LF2_ERR_DEVICE, "plan setup: %s", hipGetErrorString(e));
    }
    if (st == LF2_OK && (flags & LF2_PLAN_AUTOTUNE)) st = autotune(p);
    if (st != LF2_OK) {
        lf2_plan_destroy(p);
        return st;
    }
    *out = p;
    return LF2_OK;
}

lf2_status lf2_plan_get_tuning(lf2_plan p, int32_t axis, int32_t *variant, int32_t *chunk,
                               double *us_default, double *us_tuned)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (axis < 0 || axis > 3) return fail(LF2_ERR_INVALID_ARG, "axis %d is not 0, 1, 2 or 3", axis);
    if (axis == 3) {
        if (variant) *variant = p->fvar;
        if (chunk) *chunk = 16;
        if (us_default) *us_default = -1.0;
        if (us_tuned) *us_tuned = -1.0;
        return LF2_OK;
    }
    if (axis == 0) {
        if (variant) *variant = p->gen[0] ? -1 : p->xx;
        if (chunk) *chunk = 0;
        if (us_default) *us_default = p->tune_us[0][0];
        if (us_tuned) *us_tuned = p->tune_us[0][1];
        return LF2_OK;
    }
    if (variant) *variant = p->gen[axis] ? -1 : p->svar[axis];
    if (chunk) *chunk = p->schunk[axis];
    if (us_default) *us_default = p->tune_us[axis][0];
    if (us_tuned) *us_tuned = p->tune_us[axis][1];
    return LF2_OK;
}

lf2_status lf2_plan_get_schedule(lf2_plan p, int32_t axis, int32_t radices[15], int32_t *nst,
                                 int32_t *runtime)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (axis < 0 || axis > 2) return fail(LF2_ERR_INVALID_ARG, "axis %d is not 0, 1 or 2", axis);
    int n = 0;
    int r[kGenMaxStages] = {};
    if (p->gen[axis]) {
        n = p->sched[axis].n;
        for (int i = 0; i < n; ++i) r[i] = p->sched[axis].r[i];
    } else {
        // the factors of the compiled kernels' stages (lf2_device.hpp)
        const lf2::RadixPlan rp = lf2::radix_plan(p->len[axis]);
        n = rp.nf;
        for (int i = 0; i < n && i < kGenMaxStages; ++i) r[i] = rp.f[i];
    }
    if (nst) *nst = n;
    if (runtime) *runtime = p->gen[axis] ? 1 : 0;
    if (radices)
        for (int i = 0; i < kGenMaxStages; ++i) radices[i] = i < n ? r[i] : 0;
    return LF2_OK;
}

lf2_status lf2_plan_set_schedule(lf2_plan p, int32_t axis, const int32_t *radices, int32_t nstages)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (axis < 0 || axis > 2) return fail(LF2_ERR_INVALID_ARG, "axis %d is not 0, 1 or 2", axis);
    if (nstages < 0 || nstages > kGenMaxStages || (nstages > 0 && !radices))
        return fail(LF2_ERR_INVALID_ARG, "bad schedule (%d stages)", nstages);
    GSched sc{};
    sc.n = nstages;
    for (int i = 0; i < nstages; ++i) sc.r[i] = radices[i];
    if (!sched_valid(sc, p->len[axis]))
        return fail(LF2_ERR_INVALID_ARG,
                    "radices must each be 2, 3, 4, 5, 8 or 16 with product %d", p->len[axis]);
    if (axis == 0 && !p->gen_only[0])
        return fail(LF2_ERR_UNSUPPORTED, "the x pass of length %d runs compiled kernels only",
                    p->len[0]);
    if (axis > 0 && gs_cols(p, p->len[axis], 0) < 1)
        return fail(LF2_ERR_UNSUPPORTED, "line length %d does not fit a tile", p->len[axis]);
    p->sched[axis] = sc;
    p->gen[axis] = true;
    p->nat[axis] = false;
    if (axis < 2) p->plane = false;  // the pass that was asked for
    return LF2_OK;
}

lf2_status lf2_plan_set_tuning(lf2_plan p, int32_t axis, int32_t variant, int32_t chunk)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (axis == 0) {
        if (variant < 0 || variant > 2) return fail(LF2_ERR_INVALID_ARG, "variant %d outside [0, 2]", variant);
        if (p->gen_only[0])
            return fail(LF2_ERR_UNSUPPORTED, "no compiled kernels for line length %d", p->len[0]);
        const bool was_gen = p->gen[0];
        p->gen[0] = false;  // the compiled kernels again
        if (variant && !x_lane_exchange_ok(p)) {
            p->gen[0] = was_gen;
            return fail(LF2_ERR_UNSUPPORTED,
                        "lane exchange needs c2c rows of 64 points and one component");
        }
        p->xx = variant;
        p->plane = false;  // the pass that was asked for
        return LF2_OK;
    }
    if (axis == 3) {
        if (variant < 0 || variant > 1) return fail(LF2_ERR_INVALID_ARG, "variant %d outside [0, 1]", variant);
        if (variant == 1 && !fused_reg_supported(p->len[2]))
            return fail(LF2_ERR_UNSUPPORTED, "no register tile for the fused pass over %d points",
                        p->len[2]);
        p->fvar = variant;
        return LF2_OK;
    }
    if (axis != 1 && axis != 2) return fail(LF2_ERR_INVALID_ARG, "axis %d is not 0, 1, 2 or 3", axis);
    if (variant < 0 || variant > 7) return fail(LF2_ERR_INVALID_ARG, "variant %d outside [0, 7]", variant);
    if (chunk < 1 || chunk > 1024) return fail(LF2_ERR_INVALID_ARG, "chunk %d outside [1, 1024]", chunk);
    if (p->gen_only[axis])
        return fail(LF2_ERR_UNSUPPORTED, "no compiled kernels for line length %d", p->len[axis]);
    if ((variant & 1) && !s_wide_supported(p->len[axis]))
        return fail(LF2_ERR_UNSUPPORTED, "no wide tiles for line length %d", p->len[axis]);
    if ((variant & 4) && ((variant & 1) || !s_reg_supported(p->len[axis])))
        return fail(LF2_ERR_UNSUPPORTED, "no register tile for line length %d (or with wide tiles)",
                    p->len[axis]);
    p->svar[axis] = p->svar_b[axis] = variant;
    p->schunk[axis] = chunk;
    p->gen[axis] = false;  // the compiled kernels again
    if (axis == 1) p->plane = false;  // the pass that was asked for
    return LF2_OK;
}

lf2_status lf2_plan_destroy(lf2_plan p)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    for (void *ptr : p->allocs) (void)hipFree(ptr);
    delete p;
    return LF2_OK;
}

lf2_status lf2_fft_kspace(lf2_plan p, int64_t ksize[3], int64_t kstride[3])
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (ksize) {
        ksize[0] = p->nxk;
        ksize[1] = p->n[1];
        ksize[2] = p->n[2];
    }
    if (kstride) {
        kstride[0] = p->nc;
        if (p->klay == 2) {  // c2c (k_z, k_x, k_y): [N1][N0][N2]
            kstride[0] = p->nc * p->n[2];
            kstride[1] = p->nc * p->n[2] * p->n[0];
            kstride[2] = p->nc;
        } else {
            kstride[1] = p->klay == 1 ? p->nc * p->nxk * p->n[2] : p->nc * p->nxk;
            kstride[2] = p->klay == 1 ? p->nc * p->nxk : p->nc * p->nxk * p->n[1];
        }
    }
    return LF2_OK;
}

lf2_status lf2_plan_workspace_bytes(lf2_plan p, size_t *bytes)
{
    if (!p || !bytes) return fail(LF2_ERR_INVALID_ARG, "NULL argument");
    *bytes = ws_layout(p, true, kMaxBins, true).total;
    return LF2_OK;
}

lf2_status lf2_plan_set_workspace(lf2_plan p, void *dev_ptr, size_t bytes)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (dev_ptr && ((uintptr_t)dev_ptr % 256))
        return fail(LF2_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
    p->own_ws = dev_ptr;
    p->own_ws_bytes = dev_ptr ? bytes : 0;
    return LF2_OK;
}

lf2_status lf2_fft_execute(lf2_plan p, lf2_direction dir, const void *in, void *out, void *stream)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (dir != LF2_FORWARD && dir != LF2_BACKWARD) return fail(LF2_ERR_INVALID_ARG, "bad direction %d", (int)dir);
    lf2_status st;
    if ((st = check_ptr(in, "in", 8)) || (st = check_ptr(out, "out", 8))) return st;
    if (in == out && !p->inplace)
        return fail(LF2_ERR_UNSUPPORTED, "in == out needs a plan made with LF2_IN_PLACE");
    if ((st = check_device(p))) return st;
    hipStream_t s = (hipStream_t)stream;
    if (p->kind == LF2_R2C && dir == LF2_FORWARD) {
        if (p->klay == 1 && in == out) {
            // in place in the paper's order: the x pass moves row (y, z) to
            // another row's place, so it writes the workspace and the y pass
            // brings the spectrum back
            WsLayout L = ws_layout(p, true, 0, false);
            char *ws;
            if ((st = get_workspace(p, L.total, &ws))) return st;
            void *W = ws + L.w;
            if ((st = run_x(p, 0, -1, x_args(p, in, W, true, false, true), s))) return st;
            if ((st = run_strided(p, 1, -1, s_args(p, 1, W, out, EPI_STORE), kStridedGridCap, s, nullptr))) return st;
        } else {
            if ((st = run_xy(p, 0, -1, x_args(p, in, out, true, false, true), out, s, p->plane))) return st;
        }
        return run_strided(p, 2, -1, s_args(p, 2, out, out, EPI_STORE), kStridedGridCap, s, nullptr);
    }
    if (p->kind == LF2_R2C) {
        WsLayout L = ws_layout(p, true, 0, false);
        char *ws;
        if ((st = get_workspace(p, L.total, &ws))) return st;
        void *W = ws + L.w;
        if ((st = run_strided(p, 2, +1, s_args(p, 2, in, W, EPI_STORE), kStridedGridCap, s, nullptr))) return st;
        return run_xy(p, 1, +1, x_args(p, W, out, false, true, true), W, s, p->plane);
    }
    // c2c: x and y of a plane, then z, forward; the reverse, backward.  The
    // intermediate is out, or the workspace where out has another layout (the
    // paper's (k_z, k_x, k_y) order: the z pass stores or loads transposed) or
    // a halo (backward)
    const int sg = (int)dir;
    void *W = out;
    if (p->klay == 2 || (dir == LF2_BACKWARD && p->halo != 0)) {
        WsLayout L = ws_layout(p, true, 0, false);
        char *ws;
        if ((st = get_workspace(p, L.total, &ws))) return st;
        W = ws + L.w;
    }
    auto zpass = [&](const void *src, void *dst) {
        if (p->klay == 2)
            return run_strided(p, 2, sg,
                               t_args(p, src, dst, EPI_STORE | (sg < 0 ? EPI_TSTORE : EPI_TLOAD)),
                               kStridedGridCap, s, nullptr);
        return run_strided(p, 2, sg, s_args(p, 2, src, dst, EPI_STORE), kStridedGridCap, s, nullptr);
    };
    if (dir == LF2_FORWARD) {
        if ((st = run_xy(p, 2, sg, x_args(p, in, W, true, false, false), W, s, p->plane))) return st;
        return zpass(W, out);
    }
    if ((st = zpass(in, W))) return st;
    return run_xy(p, 2, sg, x_args(p, W, out, false, true, false), W, s, p->plane);
}

}  // extern "C"

namespace lf2 {
namespace host {

size_t poisson_ws_bytes(const lf2_plan_s *p, int32_t nbins, bool parseval)
{
    const int nb = nbins > 0 ? nbins : (parseval ? 1 : 0);
    return ws_layout(p, true, nb, parseval).total;
}

// Poisson solve on `stream`; ws_given (nullable) is a workspace of at least
// poisson_ws_bytes bytes reserved for this call, else the plan's workspace.
lf2_status poisson_impl(lf2_plan p, const float *rho, float *phi, double dx, uint32_t flags,
                        int32_t nbins, double *d_pk, double *d_kmean, double *d_count,
                        double *d_parseval, hipStream_t stream, char *ws_given,
                        size_t ws_given_bytes, bool noalloc, const PoissonTables *tabs)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (p->kind != LF2_R2C || p->nc != 1)
        return fail(LF2_ERR_UNSUPPORTED, "Poisson needs an r2c plan with ncomp = 1");
    lf2_status st;
    if ((st = check_ptr(rho, "rho", 4)) || (st = check_ptr(phi, "phi", 4))) return st;
    if ((const void *)rho == (const void *)phi && !p->inplace)
        return fail(LF2_ERR_INVALID_ARG, "rho and phi alias: needs a plan made with LF2_IN_PLACE");
    if (!(dx > 0.0) || !std::isfinite(dx)) return fail(LF2_ERR_INVALID_ARG, "dx must be > 0");
    if (flags & ~(uint32_t)(LF2_POISSON_DISCRETE_K2 | LF2_PK_OF_PHI))
        return fail(LF2_ERR_INVALID_ARG, "unknown Poisson flags 0x%x", flags);
    if ((st = check_bins(p, nbins))) return st;
    if (d_parseval && (flags & LF2_PK_OF_PHI))
        return fail(LF2_ERR_INVALID_ARG, "Parseval sums are defined for rho; drop LF2_PK_OF_PHI");
    if ((st = check_device(p))) return st;
    hipStream_t s = (hipStream_t)stream;
    const bool parseval = d_parseval != nullptr;
    const int nb = nbins > 0 ? nbins : (parseval ? 1 : 0);
    // bins and Parseval sums are FP64 sums of the forward spectrum: the plane
    // kernel makes it where it gives the two passes' bits, with bins and
    // without, so that phi does not depend on what else is asked for
    bool plane = p->plane && p->plane_bits;
    WsLayout L = ws_layout(p, true, nb, parseval, plane);
    const size_t room = ws_given ? ws_given_bytes : p->own_ws ? p->own_ws_bytes : L.total;
    if (plane && room < L.total) {
        // a workspace sized for the two passes' sums of squares: run those
        plane = false;
        L = ws_layout(p, true, nb, parseval);
    }
    char *ws;
    if (ws_given) {
        if (ws_given_bytes < L.total)
            return fail(noalloc ? LF2_ERR_UNSUPPORTED : LF2_ERR_INVALID_ARG,
                        "workspace of %zu bytes < %zu needed", ws_given_bytes, L.total);
        ws = ws_given;
    } else if (noalloc) {
        return fail(LF2_ERR_INVALID_ARG, "no workspace for a call that must not allocate");
    } else if ((st = get_workspace(p, L.total, &ws))) {
        return st;
    }
    void *W = ws + L.w;
    const double *k2[3];
    ShellEntry sh{};
    if (tabs) {
        for (int i = 0; i < 3; ++i) k2[i] = tabs->k2[i];
        sh = tabs->sh;
        if (nb > 0 && sh.nbins != nb) return fail(LF2_ERR_INVALID_ARG, "shell table of another bin count");
    } else {
        if ((st = get_k2(p, dx, (flags & LF2_POISSON_DISCRETE_K2) ? 1 : 0, s, k2, noalloc))) return st;
        if (nb > 0 && (st = get_shell(p, nb, s, &sh, noalloc))) return st;
    }

    XArgs xa = x_args(p, rho, W, true, false, true);
    if (parseval) xa.sumsq = (double *)(ws + L.sq);
    if ((st = run_xy(p, 0, -1, xa, W, s, plane))) return st;
    int epi = EPI_STORE | EPI_POISSON;
    if (nb > 0) epi |= (flags & LF2_PK_OF_PHI) ? EPI_PK_AFTER : EPI_PK;
    SArgs za = s_args(p, 2, W, W, epi);
    for (int i = 0; i < 3; ++i) za.mt.k2[i] = k2[i];
    set_k2_units(za.mt, p, dx, (flags & LF2_POISSON_DISCRETE_K2) ? 1 : 0);
    int grid = 0;
    if (nb > 0) {
        use_shell(za.mt, sh);
        za.partial = (double *)(ws + L.part);
    }
    if ((st = run_strided(p, 2, -1, za, nb > 0 ? kPkGrid : kStridedGridCap, s, &grid))) return st;
    if ((st = run_xy(p, 1, +1, x_args(p, W, phi, false, true, true), W, s, p->plane))) return st;
    if (nb > 0) {
        const double vscale = (flags & LF2_PK_OF_PHI) ? (double)p->ntot * (double)p->ntot : 1.0;
        const bool user_bins = nbins > 0;
        if ((st = pk_tail(p, sh, (const double *)(ws + L.part), grid, dx, vscale,
                          user_bins ? d_pk : nullptr, user_bins ? d_kmean : nullptr,
                          user_bins ? d_count : nullptr, d_parseval,
                          parseval ? (const double *)(ws + L.sq) : nullptr,
                          !parseval ? 0 : plane ? p->n[2] : x_grid_blocks(p), s)))
            return st;
    }
    return LF2_OK;
}

}  // namespace host
}  // namespace lf2

extern "C" {

lf2_status lf2_poisson_solve(lf2_plan p, const float *rho, float *phi, double dx, uint32_t flags,
                             int32_t nbins, double *d_pk, double *d_kmean, double *d_count,
                             double *d_parseval, void *stream)
{
    return poisson_impl(p, rho, phi, dx, flags, nbins, d_pk, d_kmean, d_count, d_parseval,
                        (hipStream_t)stream, nullptr, 0);
}

}  // extern "C"

// ------------------------------------------------ static scratch (no allocation)
// Workspace of lf2_poisson_solve_noalloc: one array per device, held by the
// code object for the life of the process.  In host code `scratch` names a
// host-side stand-in, not device memory: only the address that
// hipGetSymbolAddress returns on a device is used (kernel arguments), and it
// is looked up once per device with that device current.
static __device__ __align__(256) char scratch[LF2_NOALLOC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
char *g_scratch_ptr[kMaxDevices] = {};

lf2_status scratch_on(int dev, char **out)
{
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(LF2_ERR_DEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                        hipGetErrorString(e));
        g_scratch_ptr[dev] = (char *)ptr;
    }
    *out = g_scratch_ptr[dev];
    return LF2_OK;
}
}  // namespace

extern "C" {

lf2_status lf2_poisson_solve_noalloc(lf2_plan p, const float *rho, float *phi, double dx,
                                     uint32_t flags, int32_t nbins, double *d_pk,
                                     double *d_kmean, double *d_count, double *d_parseval,
                                     void *stream)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    lf2_status st;
    if ((st = check_device(p))) return st;
    char *ws = nullptr;
    if ((st = scratch_on(p->device, &ws))) return st;
    prof::t_quiet = true;
    st = poisson_impl(p, rho, phi, dx, flags, nbins, d_pk, d_kmean, d_count, d_parseval,
                      (hipStream_t)stream, ws, LF2_NOALLOC_SCRATCH_BYTES, true);
    prof::t_quiet = false;
    return st;
}

lf2_status lf2_power_spectrum(lf2_plan p, const void *field, int32_t field_is_kspace, int32_t nbins,
                              double dx, double *d_pk, double *d_kmean, double *d_count,
                              void *stream)
{
    if (!p) return fail(LF2_ERR_INVALID_ARG, "plan is NULL");
    if (p->nc != 1) return fail(LF2_ERR_UNSUPPORTED, "power spectrum needs ncomp = 1");
    lf2_status st;
    if ((st = check_ptr(field, "field", field_is_kspace || p->kind == LF2_C2C ? 8 : 4))) return st;
    if (nbins < 1) return fail(LF2_ERR_INVALID_ARG, "nbins %d < 1", nbins);
    if ((st = check_bins(p, nbins))) return st;
    if (!(dx > 0.0) || !std::isfinite(dx)) return fail(LF2_ERR_INVALID_ARG, "dx must be > 0");
    if ((st = check_device(p))) return st;
    hipStream_t s = (hipStream_t)stream;
    WsLayout L = ws_layout(p, !field_is_kspace, nbins, false);
    char *ws;
    if ((st = get_workspace(p, L.total, &ws))) return st;
    ShellEntry sh{};
    if ((st = get_shell(p, nbins, s, &sh))) return st;
    double *part = (double *)(ws + L.part);
    int grid = 0;
    if (field_is_kspace) {
        ModeTables mt = base_tables(p);
        use_shell(mt, sh);
        const int t = prof::begin("k_pk_kspace", (double)spectrum_bytes(p), s);
        int64_t kst[3];
        (void)lf2_fft_kspace(p, nullptr, kst);
        hipError_t e = launch_pk_kspace(field, (int)p->n[1], (int)p->n[2], kst[0], kst[1], kst[2], mt,
                                        part, kPkGrid, s, &grid);
        prof::end(t, s);
        LF2_HIP(e);
    } else {
        void *W = ws + L.w;
        const int which = p->kind == LF2_R2C ? 0 : 2;
        const XArgs xa = x_args(p, field, W, true, false, which == 0);
        if ((st = run_xy(p, which, -1, xa, W, s, p->plane && p->plane_bits))) return st;
        SArgs za = s_args(p, 2, W, W, EPI_PK);
        use_shell(za.mt, sh);
        za.partial = part;
        if ((st = run_strided(p, 2, -1, za, kPkGrid, s, &grid))) return st;
    }
    return pk_tail(p, sh, part, grid, dx, 1.0, d_pk, d_kmean, d_count, nullptr, nullptr, 0, s);
}

}  // extern "C"
