// lf2_kernels.hpp -- pass kernels of the 3-D FFT (gfx950).
//
// Every pass is written as a per-tile device function that works in an LDS
// area handed to it by the caller.  The standalone kernels below run one
// pass over one field; the batch kernels (lf2_kbatch.hip) run the same tile
// functions over the tiles of many fields, one launch per (pass, length).
//
// x pass  : lines along dimension 0 are contiguous in memory.  A tile is RB
//           rows (all components of each row).  r2c packs N0 reals as N0/2
//           complex values, transforms and splits the result into Nh bins;
//           c2r does the reverse.  Dense tiles are read as one run of
//           16-byte loads into LDS; other one-component rows with even
//           element offsets go as complex values straight into the first
//           Stockham stage, and interleaved components of real fields (or
//           odd halo offsets) as float pairs.
// strided : lines along dimension 1 or 2 have a large stride; consecutive
//           columns are adjacent in memory.  A tile is B adjacent columns x
//           L points: loaded row by row (B * 8 bytes contiguous per row)
//           straight into the first stage, transformed in LDS with lanes
//           walking adjacent columns, stored from the last stage.  This
//           replaces the paper's rod transposes (the data never leaves its
//           place; the tile is the transpose).  Epilogues on the last axis:
//           power-spectrum binning and the Poisson scale followed by the
//           backward transform.
#pragma once
#include "lf2_device.hpp"
#include "lf2_internal.hpp"

namespace lf2 {

constexpr int kXThreads = 256;

// Rows per x-pass tile: about 4096 * (NT / 256) complex values of LDS, at
// most 256 rows.
__host__ __device__ constexpr int x_rb(int L, int NC, int NT = kXThreads)
{
    return ((4096 / L) / NC * (NT / 256)) < 1
               ? 1
               : (((4096 / L) / NC * (NT / 256)) > 256 ? 256 : ((4096 / L) / NC * (NT / 256)));
}
__host__ __device__ constexpr size_t al16(size_t b) { return (b + 15) & ~(size_t)15; }

// LDS bytes of a narrow strided tile: its columns and the twiddle table.
__host__ __device__ constexpr size_t s_bytes(int L)
{
    return al16(al16(sizeof(c32) * L * s_b(L)) + sizeof(c32) * L);
}

template <int RB>
__device__ __forceinline__ int rows_valid(const XArgs &a, int64_t r0)
{
    const int64_t left = a.nrows - r0;
    return left < RB ? (int)left : RB;
}

// FP64 block sum of v into *dst (thread 0 writes).
template <int NT>
__device__ __forceinline__ void block_sum_f64(double v, double *dst, double *scratch)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) scratch[wid] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0;
        for (int w = 0; w < NT / 64; ++w) t += scratch[w];
        *dst = t;
    }
}

// Twiddle tables into LDS (callers wait at a barrier before use).
__device__ __forceinline__ void load_table(c32 *dst, const void *src, int n, int tid, int nt)
{
    const c32 *g = (const c32 *)src;
    for (int i = tid; i < n; i += nt) dst[i] = g[i];
}

// A table of N values on its way to LDS through the threads' registers: its
// loads are issued beside a tile's own, so that both are waited for once.
// (x passes over 512^3 with three components, us: r2c 710 -> 669, c2r 681 ->
// 641; 256^3 c2r 25.6 -> 24.2.)
template <int N, int NT>
struct TableRegs {
    static constexpr int K = (N + NT - 1) / NT;
    c32 w[K];
    __device__ __forceinline__ void load(const void *src, int tid)
    {
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (N % NT == 0 || tid + i * NT < N) w[i] = ((const c32 *)src)[tid + i * NT];
    }
    __device__ __forceinline__ void store(c32 *dst, int tid) const
    {
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (N % NT == 0 || tid + i * NT < N) dst[tid + i * NT] = w[i];
    }
};

// Forward lines whose table (and x rows' offsets, in LDS) stay ahead of loads
// that feed the first stage: behind them the compiler rounds the 16-point
// butterfly of 16 3 and 16 5 (2^a) points another way, and P(k) of a field
// would move in its ninth digit.
__host__ __device__ constexpr bool table_first(int L)
{
    const RadixPlan p = radix_plan(L);
    return p.nodd == 1 && p.f[0] == 16;
}

// Row offsets of a tile's first nv rows into LDS.
template <int RB, int NT>
__device__ __forceinline__ void fill_rows(int64_t *ib, const RowAt &at, int nv, int tid)
{
    for (int i = tid; i < RB; i += NT) ib[i] = at(i < nv ? i : nv - 1);
}

// The real x tiles' hooks: the sum of squares of the input, where it is asked
// for, and the tables' way on to LDS, with a barrier where the first stage
// reads them (kPaired).
template <class Tabs>
struct RealHook {
    double *ss;
    bool sum;
    Tabs tabs;
    template <int R>
    __device__ __forceinline__ void values(const c32 (&v)[R]) const
    {
        if (!sum) return;
#pragma unroll
        for (int r = 0; r < R; ++r) *ss += (double)v[r].x * v[r].x + (double)v[r].y * v[r].y;
    }
    __device__ __forceinline__ void loaded() const { tabs(); }
};
template <class Tabs>
struct TabHook {
    Tabs tabs;
    template <int R>
    __device__ __forceinline__ void values(const c32 (&)[R]) const {}
    __device__ __forceinline__ void loaded() const { tabs(); }
};
template <class Tabs>
__device__ __forceinline__ TabHook<Tabs> tab_hook(Tabs t)
{
    return TabHook<Tabs>{t};
}
template <class Tabs>
__device__ __forceinline__ RealHook<Tabs> real_hook(double &ss, bool sum, Tabs t)
{
    return RealHook<Tabs>{&ss, sum, t};
}

// =================================================================== x tiles
// tab of a tile function: the block's first tile, which fetches the tables
// itself, beside its own loads (else they are in LDS).

// ---- general r2c (interleaved components, any float offsets): the first
// stage loads component c's packed point n = (f[2n][c], f[2n + 1][c]) as two
// floats straight from the row; one padded LDS line per (row, component)
template <int M, int NC, int NT>
struct XR2CGen {
    static constexpr int RB = x_rb(M, NC, NT), NL = RB * NC, LP = row_pitch(M),
                         NH = M + 1;
    // one component alone feeds P(k), whose bits the table's place decides
    static constexpr bool kTableFirst = NC == 1 && table_first(M);
    static constexpr size_t O_BUF = 0, O_TW = al16(O_BUF + sizeof(c32) * NL * LP),
                            O_TWP = al16(O_TW + sizeof(c32) * M),
                            O_RED = al16(O_TWP + sizeof(c32) * NH),
                            O_OB = al16(O_RED + 8 * (NT / 64)), O_IB = O_OB + 8 * RB,
                            BYTES = O_IB + (kTableFirst ? 8 * RB : 0);
    static __device__ void tables(const XArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, M, tid, NT);
        load_table((c32 *)(sm + O_TWP), a.tw_post, NH, tid, NT);
    }
    // sumsq: where to put this tile's FP64 sum of squares (nullptr: skip)
    static __device__ void tile(const XArgs &a, int64_t blk, char *sm, int tid, double *sumsq,
                                bool tab = false)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW), *twp = (const c32 *)(sm + O_TWP);
        const int64_t r0 = blk * RB;
        const RowAt in_at = row_at(a.in_off, a.in_row, a.in_plane, a.n1, r0);
        const RowAt out_at = row_at(a.out_off, a.out_row, a.out_plane, a.n1, r0);
        const int nv = rows_valid<RB>(a, r0);
        // the first stage reads each component's packed pairs straight from
        // the real rows (two float loads per point; no alignment needed)
        double ss = 0.0;
        // the store below looks rows up for every value, so their offsets are
        // kept (computed there, 96 x 192 x 128 with six components 35 -> 39 us)
        int64_t *ob = (int64_t *)(sm + O_OB);
        if constexpr (kTableFirst) {
            if (tab) tables(a, sm, tid);
            int64_t *ib = (int64_t *)(sm + O_IB);
            fill_rows<RB, NT>(ib, in_at, nv, tid);
            fill_rows<RB, NT>(ob, out_at, nv, tid);
            __syncthreads();
            row_fft<M, -1, RB, NC, LP, NT, true, false, 0, 1, true, true>(
                buf, (const c32 *)a.in, nullptr, RowTable{ib}, RowTable{ib}, nv, tw, tid,
                real_hook(ss, sumsq != nullptr, [] {}));
        } else {
            TableRegs<M, NT> wt;
            TableRegs<NH, NT> wp;
            if (tab) {
                wt.load(a.tw, tid);
                wp.load(a.tw_post, tid);
            }
            row_fft<M, -1, RB, NC, LP, NT, true, false, 0, 1, true, true>(
                buf, (const c32 *)a.in, nullptr, in_at, out_at, nv, tw, tid,
                real_hook(ss, sumsq != nullptr, [&] {
                    fill_rows<RB, NT>(ob, out_at, nv, tid);
                    if (!tab) return;
                    wt.store((c32 *)(sm + O_TW), tid);
                    wp.store((c32 *)(sm + O_TWP), tid);
                    if (kPaired<M>) __syncthreads();  // else the first stage reads no table
                }));
        }
        if (sumsq) block_sum_f64<NT>(ss, sumsq, (double *)(sm + O_RED));
        // X[k] = fe + W^k fo and X[M-k] = conj(fe - W^k fo) per component;
        // work item (row, k, component), component fastest
        c32 *out = (c32 *)a.out;
        constexpr int HALF = M / 2 + 1;
        constexpr int NI = RB * HALF * NC;
#pragma unroll
        for (int i = 0; i < (NI + NT - 1) / NT; ++i) {
            const int idx = tid + i * NT;
            if (idx < NI) {
                const int c = idx % NC, t = idx / NC;
                const int k = t % HALF, l = t / HALF;
                if (l < nv) {
                    const c32 *line = buf + (l * NC + c) * LP;
                    const c32 z = line[lpad(k)];
                    const c32 zc = conjg(line[lpad(k == 0 ? 0 : M - k)]);
                    const c32 fe = scl(add(z, zc), 0.5f);
                    const c32 d = sub(z, zc);
                    const c32 fo = c32{0.5f * d.y, -0.5f * d.x};  // (z - zc) / (2i)
                    const c32 wf = mul(twp[k], fo);
                    c32 *orow = out + ob[l] + c;
                    gstore<true>(orow + k * NC, add(fe, wf));
                    if (2 * k != M) gstore<true>(orow + (M - k) * NC, conjg(sub(fe, wf)));
                }
            }
        }
        __syncthreads();
    }
};

// ---- general c2r (interleaved components, any float offsets): bins through
// LDS, and the last stage stores each packed point as two floats
template <int M, int NC, int NT>
struct XC2RGen {
    static constexpr int RB = x_rb(M, NC, NT), NL = RB * NC, LP = row_pitch(M + 1), NH = M + 1;
    static constexpr size_t O_BUF = 0, O_TW = al16(O_BUF + sizeof(c32) * NL * LP),
                            O_TWP = al16(O_TW + sizeof(c32) * M),
                            O_OB = al16(O_TWP + sizeof(c32) * NH), BYTES = O_OB + 8 * RB;
    static __device__ void tables(const XArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, M, tid, NT);
        load_table((c32 *)(sm + O_TWP), a.tw_post, NH, tid, NT);
    }
    // Whole output rows leave as 16-byte nontemporal stores when every row
    // starts 16-byte aligned and holds a multiple of 4 floats.
    static __device__ bool vec_out(const XArgs &a)
    {
        return (2 * M * NC) % 4 == 0 && ((uintptr_t)a.out & 15) == 0 && a.out_off % 4 == 0 &&
               a.out_row % 4 == 0 && a.out_plane % 4 == 0;
    }
    // Real rows from the LDS lines: float x NC + c of row l is part x & 1 of
    // point x >> 1 of line l NC + c.
    static __device__ void store_rows(const XArgs &a, const c32 *buf, const RowTable &out_at, int nv,
                                      int tid)
    {
        typedef float nf4 __attribute__((ext_vector_type(4)));
        constexpr int W4 = 2 * M * NC / 4;  // 16-byte words per row
        const float *fb = (const float *)buf;
        float *out = (float *)a.out;
        for (int e = tid; e < nv * W4; e += NT) {
            const int l = e / W4, f0 = 4 * (e - l * W4);
            float w[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int f = f0 + u, x = f / NC, c = f - x * NC;
                w[u] = fb[2 * ((l * NC + c) * LP + lpad(x >> 1)) + (x & 1)];
            }
            nf4 v;
            v.x = w[0];
            v.y = w[1];
            v.z = w[2];
            v.w = w[3];
            __builtin_nontemporal_store(v, (nf4 *)(out + out_at(l)) + (e - l * W4));
        }
    }
    static __device__ void tile(const XArgs &a, int64_t blk, char *sm, int tid, bool tab = false)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW), *twp = (const c32 *)(sm + O_TWP);
        const int64_t r0 = blk * RB;
        const RowAt in_at = row_at(a.in_off, a.in_row, a.in_plane, a.n1, r0);
        int64_t *ob = (int64_t *)(sm + O_OB);  // offsets of the rows to store, kept
        const RowTable out_at{ob};
        TableRegs<M, NT> wt;
        TableRegs<NH, NT> wp;
        if (tab) {
            wt.load(a.tw, tid);
            wp.load(a.tw_post, tid);
        }
        auto tabs = [&](bool sync) {
            if (!tab) return;
            wt.store((c32 *)(sm + O_TW), tid);
            wp.store((c32 *)(sm + O_TWP), tid);
            if (sync) __syncthreads();
        };
        const c32 *in = (const c32 *)a.in;
        constexpr int NI = RB * NH * NC;
        const int nv = rows_valid<RB>(a, r0);
        // value e of the tile's rows (row-major, component fastest) -> LDS
        auto put = [&](int e, c32 v) {
            const int row = e / (NH * NC), rem = e - row * (NH * NC);
            const int k = rem / NC, c = rem - k * NC;
            buf[(row * NC + c) * LP + lpad(k)] = v;
        };
        const c32 *src = in + in_at(0);
        if (a.in_row == NH * NC && a.in_plane == (int64_t)a.n1 * NH * NC &&
            ((uintptr_t)src & 7) == 0) {
            // dense half spectrum: the tile's rows are one contiguous run,
            // read with 16-byte loads from the first 16-byte boundary on
            // (all of a thread's loads are issued before the first LDS write)
            typedef float nf4 __attribute__((ext_vector_type(4)));
            constexpr int NW = (NI / 2 + NT - 1) / NT;
            const int e0 = ((uintptr_t)src & 15) ? 1 : 0;
            const nf4 *s4 = (const nf4 *)(src + e0);
            const int cnt = nv * NH * NC;
            const int np = (cnt - e0) / 2;
            nf4 w[NW];
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int e = tid + i * NT;
                if (e < np) w[i] = __builtin_nontemporal_load(s4 + e);
            }
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int e = tid + i * NT;
                if (e < np) {
                    put(e0 + 2 * e, c32{w[i].x, w[i].y});
                    put(e0 + 2 * e + 1, c32{w[i].z, w[i].w});
                }
            }
            if (tid == 0 && e0 && cnt > 0) put(0, src[0]);
            if (tid == 0 && e0 + 2 * np < cnt) put(cnt - 1, src[cnt - 1]);
            for (int e = cnt + tid; e < NI; e += NT) put(e, c32{0.f, 0.f});
        } else {
#pragma unroll
            for (int i = 0; i < (NI + NT - 1) / NT; ++i) {
                const int idx = tid + i * NT;
                if (idx < NI) {
                    const int row = idx / (NH * NC);
                    put(idx, row < nv ? gload<true>(in + in_at(row) + (idx - row * (NH * NC)))
                                      : c32{0.f, 0.f});
                }
            }
        }
        tabs(false);
        fill_rows<RB, NT>(ob, row_at(a.out_off, a.out_row, a.out_plane, a.n1, r0), nv, tid);
        __syncthreads();
        // Z[k] = (X[k] + conj X[M-k]) + i W^{-k} (X[k] - conj X[M-k]), k < M,
        // with the imaginary parts of X[0] and X[M] dropped.
        auto zval = [&](const c32 *line, int k) {
            c32 xk = line[lpad(k)], xm = line[lpad(M - k)];
            if (k == 0) {
                xk.y = 0.f;
                xm.y = 0.f;
            }
            const c32 xmc = conjg(xm);
            const c32 sm_ = add(xk, xmc);
            const c32 d = mul(conjg(twp[k]), sub(xk, xmc));
            return c32{sm_.x - d.y, sm_.y + d.x};  // s + i d
        };
        if constexpr (kPlan<M>.n >= 2) {
            // the first inverse stage forms its inputs Z[k] from the bins in
            // LDS as it reads them (butterfly b: component b % NC, then j,
            // then row, as in the row engine), then the remaining stages
            constexpr int R = kPlan<M>.r[0], Q = M / R;
            constexpr int NBF = NL * Q, NB = (NBF + NT - 1) / NT;
            c32 v[NB][R];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int b = tid + i * NT;
                if (NBF % NT == 0 || b < NBF) {
                    const int c = b % NC, t = b / NC;
                    const int j = t % Q, q = t / Q;
                    const c32 *line = buf + (q * NC + c) * LP;
#pragma unroll
                    for (int r = 0; r < R; ++r) v[i][r] = zval(line, j + r * Q);
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int b = tid + i * NT;
                if (NBF % NT == 0 || b < NBF) {
                    const int c = b % NC, t = b / NC;
                    const int j = t % Q, q = t / Q;
                    dft_first<M, R, kPlan<M>.r1[0], +1>(v[i], tw);
                    c32 *dst = buf + (q * NC + c) * LP;
#pragma unroll
                    for (int r = 0; r < R; ++r) dst[lpad(j * R + r)] = v[i][r];
                }
            }
            __syncthreads();
            if (vec_out(a)) {
                // remaining stages in LDS, then whole rows out as 16-byte stores
                row_fft<M, +1, RB, NC, LP, NT, false, false, 1, R>(buf, nullptr, nullptr, out_at,
                                                                   out_at, nv, tw, tid);
                store_rows(a, buf, out_at, nv, tid);
            } else {
                // the last stage stores each component's pairs straight to the rows
                row_fft<M, +1, RB, NC, LP, NT, false, true, 1, R, true, true>(
                    buf, nullptr, (c32 *)a.out, out_at, out_at, nv, tw, tid);
            }
        } else {
            constexpr int NZ = NL * M;
            constexpr int NZT = (NZ + NT - 1) / NT;
            c32 zv[NZT];
#pragma unroll
            for (int i = 0; i < NZT; ++i) {
                const int idx = tid + i * NT;
                if (idx < NZ) zv[i] = zval(buf + (idx / M) * LP, idx % M);
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NZT; ++i) {
                const int idx = tid + i * NT;
                if (idx < NZ) buf[(idx / M) * LP + lpad(idx % M)] = zv[i];
            }
            __syncthreads();
            row_fft<M, +1, RB, NC, LP, NT, false, true, 0, 1, true, true>(
                buf, nullptr, (c32 *)a.out, out_at, out_at, nv, tw, tid);
        }
        __syncthreads();
    }
};

// ---- one-component fast r2c.
// X[k] = fe + W^k fo and X[M-k] = conj(fe - W^k fo), with
// fe = (Z[k] + conj Z[M-k]) / 2, fo = (Z[k] - conj Z[M-k]) / (2i).
template <int M, int NT>
struct XR2CV {
    // (rows of up to 16 points an odd pitch apart: 32 x 192 x 1024 14.6 us at a
    // pitch of 16, 13.3 at one of 17)
    static constexpr int RB = x_rb(M, 1, NT), LP = M <= 16 ? (M | 1) : row_pitch(M), NH = M + 1;
    static constexpr size_t O_BUF = 0, O_TW = al16(O_BUF + sizeof(c32) * RB * LP),
                            O_TWP = al16(O_TW + sizeof(c32) * M),
                            O_RED = al16(O_TWP + sizeof(c32) * NH),
                            O_IB = al16(O_RED + 8 * (NT / 64)),
                            BYTES = O_IB + (table_first(M) ? 8 * RB : 0);
    static __device__ void tables(const XArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, M, tid, NT);
        load_table((c32 *)(sm + O_TWP), a.tw_post, NH, tid, NT);
    }
    static __device__ void tile(const XArgs &a, int64_t blk, char *sm, int tid, double *sumsq,
                                bool tab = false)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW), *twp = (const c32 *)(sm + O_TWP);
        const int64_t r0 = blk * RB;
        const int nv = rows_valid<RB>(a, r0);
        const RowAt out_at = row_at(a.out_off, a.out_row, a.out_plane, a.n1, r0);
        TableRegs<M, NT> wt;
        TableRegs<NH, NT> wp;
        // dense rows: behind the data, not ahead of it (400^3 98 us, 112 ahead)
        auto fetch = [&] {
            if (!tab) return;
            wt.load(a.tw, tid);
            wp.load(a.tw_post, tid);
        };
        auto tabs = [&](bool sync) {
            if (!tab) return;
            wt.store((c32 *)(sm + O_TW), tid);
            wp.store((c32 *)(sm + O_TWP), tid);
            if (sync) __syncthreads();
        };
        double ss = 0.0;
        const bool dense_out = a.out_row == NH && a.out_plane == (int64_t)a.n1 * NH;
        const float *src = (const float *)a.in + a.in_off + r0 * (2 * M);
        if (M % 2 == 0 && a.in_row == 2 * M && a.in_plane == (int64_t)a.n1 * 2 * M &&
            ((uintptr_t)src & 15) == 0) {
            // Dense rows: the tile is one contiguous run of nv N0 reals, read
            // with 16-byte loads (all of a thread's loads issued first) into
            // the padded LDS lines, then transformed there.
            typedef float nf4 __attribute__((ext_vector_type(4)));
            constexpr int NW = (RB * M / 2 + NT - 1) / NT;
            const nf4 *s4 = (const nf4 *)src;
            const int np = nv * M / 2;
            auto put = [&](int e, c32 v) {
                const int l = e / M, k = e - l * M;
                buf[l * LP + lpad(k)] = v;
            };
            nf4 w[NW];
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int e = tid + i * NT;
                if (e < np) w[i] = __builtin_nontemporal_load(s4 + e);
            }
            fetch();
            tabs(false);
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int e = tid + i * NT;
                if (e < np) {
                    put(2 * e, c32{w[i].x, w[i].y});
                    put(2 * e + 1, c32{w[i].z, w[i].w});
                    if (sumsq)
                        ss += ((double)w[i].x * w[i].x + (double)w[i].y * w[i].y) +
                              ((double)w[i].z * w[i].z + (double)w[i].w * w[i].w);
                }
            }
            for (int e = nv * M + tid; e < RB * M; e += NT) put(e, c32{0.f, 0.f});
            __syncthreads();
            row_fft<M, -1, RB, 1, LP, NT, false, false>(buf, nullptr, nullptr, out_at, out_at, nv,
                                                        tw, tid);
        } else {
            // float offsets -> complex offsets
            const RowAt in_at = row_at(a.in_off / 2, a.in_row / 2, a.in_plane / 2, a.n1, r0);
            if constexpr (table_first(M)) {
                if (tab) tables(a, sm, tid);
                int64_t *ib = (int64_t *)(sm + O_IB);
                fill_rows<RB, NT>(ib, in_at, nv, tid);
                __syncthreads();
                row_fft<M, -1, RB, 1, LP, NT, true, false, 0, 1, true>(
                    buf, (const c32 *)a.in, nullptr, RowTable{ib}, RowTable{ib}, nv, tw, tid,
                    real_hook(ss, sumsq != nullptr, [] {}));
            } else {
                fetch();
                row_fft<M, -1, RB, 1, LP, NT, true, false, 0, 1, true>(
                    buf, (const c32 *)a.in, nullptr, in_at, out_at, nv, tw, tid,
                    real_hook(ss, sumsq != nullptr, [&] { tabs(kPaired<M>); }));
            }
        }
        if (sumsq) block_sum_f64<NT>(ss, sumsq, (double *)(sm + O_RED));
        // The store forms the bins from the points as it reads them: bin k of
        // line l from Z[k] and Z[M - k], indices mod M.
        c32 *out = (c32 *)a.out;
        auto bin = [&](int l, int k) {
            const c32 *line = buf + l * LP;
            const c32 z = line[lpad(k == M ? 0 : k)];
            const c32 zc = conjg(line[lpad(k == 0 || k == M ? 0 : M - k)]);
            const c32 fe = scl(add(z, zc), 0.5f);
            const c32 d = sub(z, zc);
            return add(fe, mul(twp[k], c32{0.5f * d.y, -0.5f * d.x}));
        };
        if (dense_out) {
            // dense half spectrum: the tile's rows are one contiguous run,
            // written with 16-byte nontemporal stores from the first 16-byte
            // boundary on
            typedef float nf4 __attribute__((ext_vector_type(4)));
            c32 *dst = out + a.out_off + r0 * NH;
            const int cnt = nv * NH;
            const int e0 = ((uintptr_t)dst & 15) ? 1 : 0;
            const int np = (cnt - e0) / 2;
            nf4 *d4 = (nf4 *)(dst + e0);
            for (int e = tid; e < np; e += NT) {
                const int f = e0 + 2 * e, l = f / NH, k = f - l * NH;
                const bool wrap = k == M;
                const c32 u = bin(l, k), w = bin(wrap ? l + 1 : l, wrap ? 0 : k + 1);
                nf4 v;
                v.x = u.x;
                v.y = u.y;
                v.z = w.x;
                v.w = w.y;
                __builtin_nontemporal_store(v, d4 + e);
            }
            if (tid == 0 && e0 && cnt > 0) gstore<true>(dst, bin(0, 0));
            if (tid == 0 && e0 + 2 * np < cnt) gstore<true>(dst + (cnt - 1), bin(nv - 1, M));
        } else {
            for (int e = tid; e < nv * NH; e += NT) {
                const int l = e / NH, k = e - l * NH;
                gstore<true>(out + out_at(l) + k, bin(l, k));
            }
        }
        __syncthreads();
    }
};

// ---- one-component fast c2r.
// Z[k] = (X[k] + conj X[M-k]) + i W^{-k} (X[k] - conj X[M-k]); every thread
// owns the pair (k, M-k), so the update is in place without a barrier.
template <int M, int NT>
struct XC2RV {
    static constexpr int RB = x_rb(M, 1, NT), LP = row_pitch(M + 1), NH = M + 1, HALF = M / 2 + 1;
    static constexpr size_t O_BUF = 0, O_TW = al16(O_BUF + sizeof(c32) * RB * LP),
                            O_TWP = al16(O_TW + sizeof(c32) * M),
                            BYTES = al16(O_TWP + sizeof(c32) * NH);
    static __device__ void tables(const XArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, M, tid, NT);
        load_table((c32 *)(sm + O_TWP), a.tw_post, NH, tid, NT);
    }
    static __device__ void tile(const XArgs &a, int64_t blk, char *sm, int tid, bool tab = false)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW), *twp = (const c32 *)(sm + O_TWP);
        const int64_t r0 = blk * RB;
        const RowAt in_at = row_at(a.in_off, a.in_row, a.in_plane, a.n1, r0);
        // float offsets -> complex offsets
        const RowAt out_at = row_at(a.out_off / 2, a.out_row / 2, a.out_plane / 2, a.n1, r0);
        TableRegs<M, NT> wt;
        TableRegs<NH, NT> wp;
        if (tab) {
            wt.load(a.tw, tid);
            wp.load(a.tw_post, tid);
        }
        auto tabs = [&](bool sync) {
            if (!tab) return;
            wt.store((c32 *)(sm + O_TW), tid);
            wp.store((c32 *)(sm + O_TWP), tid);
            if (sync) __syncthreads();
        };
        const int nv = rows_valid<RB>(a, r0);
        const c32 *in = (const c32 *)a.in;
        if (a.in_row == NH && a.in_plane == (int64_t)a.n1 * NH) {
            // Dense half spectrum: the tile's rows are one contiguous run of
            // nv * NH values, read with 16-byte loads when the run is 16-byte
            // aligned and placed into the padded LDS rows.
            const c32 *src = in + in_at(0);
            const int cnt = nv * NH;
            auto put = [&](int e, c32 v) {
                const int l = e / NH, k = e - l * NH;
                buf[l * LP + lpad(k)] = v;
            };
            if (((uintptr_t)src & 15) == 0) {
                // all of a thread's loads are issued before the first LDS write
                typedef float nf4 __attribute__((ext_vector_type(4)));
                constexpr int NW = (RB * NH / 2 + NT - 1) / NT;
                const nf4 *s4 = (const nf4 *)src;
                nf4 w[NW];
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    const int e = tid + i * NT;
                    if (e < cnt / 2) w[i] = __builtin_nontemporal_load(s4 + e);
                }
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    const int e = tid + i * NT;
                    if (e < cnt / 2) {
                        put(2 * e, c32{w[i].x, w[i].y});
                        put(2 * e + 1, c32{w[i].z, w[i].w});
                    }
                }
                if ((cnt & 1) && tid == 0) put(cnt - 1, src[cnt - 1]);
            } else {
                for (int e = tid; e < cnt; e += NT) put(e, src[e]);
            }
            for (int e = cnt + tid; e < RB * NH; e += NT) put(e, c32{0.f, 0.f});
        } else {
            // TPR threads per row, each walking one row: a single row offset
            // per thread, loads of a wave contiguous within each row.
            constexpr int TPR = NT / RB >= 1 ? NT / RB : 1;
            constexpr int NK = (NH + TPR - 1) / TPR;
            for (int l = tid / TPR; l < RB; l += NT / TPR) {
                const int64_t base = in_at(l);
                const bool ok = l < nv;
                const int k0 = tid % TPR;
#pragma unroll
                for (int i = 0; i < NK; ++i) {
                    const int k = k0 + i * TPR;
                    if (k < NH) buf[l * LP + lpad(k)] = ok ? in[base + k] : c32{0.f, 0.f};
                }
            }
        }
        tabs(false);
        __syncthreads();
        if constexpr (kPlan<M>.n >= 2) {
            // The first inverse stage forms its inputs Z[k] from the bins
            // X[k], X[M-k] in LDS as it reads them (every read before the
            // barrier, every write after it), then the remaining stages.
            constexpr int R = kPlan<M>.r[0], Q = M / R;
            constexpr int NBF = RB * Q, NB = (NBF + NT - 1) / NT;
            c32 v[NB][R];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int b = tid + i * NT;
                if (NBF % NT == 0 || b < NBF) {
                    const int j = b % Q, q = b / Q;
                    const c32 *line = buf + q * LP;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int k = j + r * Q;
                        c32 xk = line[lpad(k)], xm = line[lpad(M - k)];
                        if (k == 0) {
                            xk.y = 0.f;
                            xm.y = 0.f;
                        }
                        const c32 s1 = add(xk, conjg(xm));
                        const c32 d1 = mul(conjg(twp[k]), sub(xk, conjg(xm)));
                        v[i][r] = c32{s1.x - d1.y, s1.y + d1.x};
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int b = tid + i * NT;
                if (NBF % NT == 0 || b < NBF) {
                    const int j = b % Q, q = b / Q;
                    dft_first<M, R, kPlan<M>.r1[0], +1>(v[i], tw);
                    c32 *dst = buf + q * LP;
#pragma unroll
                    for (int r = 0; r < R; ++r) dst[lpad(j * R + r)] = v[i][r];
                }
            }
            __syncthreads();
            row_fft<M, +1, RB, 1, LP, NT, false, true, 1, R, true>(buf, nullptr, (c32 *)a.out, out_at,
                                                             out_at, nv, tw, tid);
        } else {
            constexpr int NP = RB * HALF;
#pragma unroll
            for (int i = 0; i < (NP + NT - 1) / NT; ++i) {
                const int idx = tid + i * NT;
                if (idx < NP) {
                    const int l = idx / HALF;
                    const int k = idx - l * HALF;
                    c32 *line = buf + l * LP;
                    c32 xk = line[lpad(k)], xm = line[lpad(M - k)];
                    if (k == 0) {
                        xk.y = 0.f;
                        xm.y = 0.f;
                    }
                    const c32 s1 = add(xk, conjg(xm));
                    const c32 d1 = mul(conjg(twp[k]), sub(xk, conjg(xm)));
                    const c32 zk = c32{s1.x - d1.y, s1.y + d1.x};
                    if (k != 0 && 2 * k != M) {
                        const c32 s2 = add(xm, conjg(xk));
                        const c32 d2 = mul(conjg(twp[M - k]), sub(xm, conjg(xk)));
                        line[lpad(M - k)] = c32{s2.x - d2.y, s2.y + d2.x};
                    }
                    line[lpad(k)] = zk;
                }
            }
            __syncthreads();
            row_fft<M, +1, RB, 1, LP, NT, false, true>(buf, nullptr, (c32 *)a.out, out_at, out_at, nv,
                                                       tw, tid);
        }
        __syncthreads();
    }
};

// ---- c2c with NC interleaved components, register-direct both ends
template <int L, int NC, int S, int NT>
struct XC2CV {
    static constexpr int RB = x_rb(L, NC, NT), LP = row_pitch(L);
    static constexpr size_t O_BUF = 0, O_TW = al16(O_BUF + sizeof(c32) * RB * NC * LP),
                            O_IB = al16(O_TW + sizeof(c32) * L), O_OB = O_IB + 8 * RB,
                            BYTES = al16(O_OB + 8 * RB);
    static __device__ void tables(const XArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, L, tid, NT);
    }
    static __device__ void tile(const XArgs &a, int64_t blk, char *sm, int tid, bool tab = false)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW);
        const int64_t r0 = blk * RB;
        const int nv = rows_valid<RB>(a, r0);
        const RowAt in_at = row_at(a.in_off, a.in_row, a.in_plane, a.n1, r0);
        const RowAt out_at = row_at(a.out_off, a.out_row, a.out_plane, a.n1, r0);
        if constexpr (S < 0) {
            // Forward, the table and the row offsets are waited for before
            // the loads: with either behind them the compiler rounds the
            // twiddle products of some rows another way, and P(k) of a field
            // would move in its ninth digit.
            if (tab) tables(a, sm, tid);
            int64_t *ib = (int64_t *)(sm + O_IB), *ob = (int64_t *)(sm + O_OB);
            fill_rows<RB, NT>(ib, in_at, nv, tid);
            fill_rows<RB, NT>(ob, out_at, nv, tid);
            __syncthreads();
            row_fft<L, S, RB, NC, LP, NT, true, true, 0, 1, true>(
                buf, (const c32 *)a.in, (c32 *)a.out, RowTable{ib}, RowTable{ob}, nv, tw, tid);
        } else {
            TableRegs<L, NT> wt;
            if (tab) wt.load(a.tw, tid);
            // the last stage's row offsets are kept where a barrier lies before it
            constexpr bool kept = kPlan<L>.n > 1;
            int64_t *ob = (int64_t *)(sm + O_OB);
            auto tabs = tab_hook([&] {
                if (kept) fill_rows<RB, NT>(ob, out_at, nv, tid);
                if (!tab) return;
                wt.store((c32 *)(sm + O_TW), tid);
                if (kPaired<L>) __syncthreads();  // else the first stage reads no table
            });
            if constexpr (kept)
                row_fft<L, S, RB, NC, LP, NT, true, true, 0, 1, true>(
                    buf, (const c32 *)a.in, (c32 *)a.out, in_at, RowTable{ob}, nv, tw, tid, tabs);
            else
                row_fft<L, S, RB, NC, LP, NT, true, true, 0, 1, true>(
                    buf, (const c32 *)a.in, (c32 *)a.out, in_at, out_at, nv, tw, tid, tabs);
        }
        __syncthreads();
    }
};

// ================================================================ binning
// Exact bin of integer squared radius q: max{b <= nbins-1 : thresh[b] <= q},
// thresh[b] = ceil(b^2 qmax / nbins^2), from an estimate corrected by
// integer comparisons against the bin's edges, so the result never depends
// on rounding.

// Bin edges (thresh[b], thresh[b + 1]) of bin b = 0..nbins as one 8-byte
// LDS entry; thresholds are < 2^32.  hi = 2^32 - 1 for the last bin (which
// also holds q = qmax) and past it.
struct BinEdge {
    uint32_t lo, hi;
};

// That bin for q < 2^32 and nbins <= 4096 from the edge table: the FP32
// estimate nbins sqrt(q / qmax) (cq = nbins^2 / qmax) is within 1e-3 of the
// exact value, so one comparison each way against the estimated bin's
// edges makes it exact.
__device__ __forceinline__ int bin_est(uint32_t q, float cq)
{
    // hardware square root (about 1 ulp; the correction absorbs it)
    return (int)__builtin_amdgcn_sqrtf((float)q * cq);  // 0..nbins
}
__device__ __forceinline__ int bin_fix(uint32_t q, int b, BinEdge e, int nbins)
{
    b += (q >= e.hi ? 1 : 0) - (q < e.lo ? 1 : 0);
    return b < nbins - 1 ? b : nbins - 1;
}
__device__ __forceinline__ int bin_edge(uint32_t q, int nbins, float cq, const BinEdge *edges)
{
    const int b = bin_est(q, cq);
    return bin_fix(q, b, edges[b], nbins);
}

// Zero the block's LDS histogram and fill its edge table.
__device__ __forceinline__ void load_edges(const ModeTables &mt, double *hist, BinEdge *edges,
                                           int tid, int nt)
{
    for (int i = tid; i <= mt.nbins; i += nt) {
        hist[i] = 0.0;
        edges[i] = BinEdge{(uint32_t)mt.thresh[i],
                           i < mt.nbins - 1 ? (uint32_t)mt.thresh[i + 1] : 0xffffffffu};
    }
}

// The same for `copies` histograms of nbins + 1 entries, one after another
// (one per wave of the block, or one for all).
__device__ __forceinline__ void hist_init(const ModeTables &mt, int copies, double *hist,
                                          BinEdge *edges, int tid, int nt)
{
    load_edges(mt, hist, edges, tid, nt);
    for (int i = mt.nbins + 1 + tid; i < copies * (mt.nbins + 1); i += nt) hist[i] = 0.0;
}

// out[i] = sum of the copies' entry i, copy 0 first (a fixed order: the
// block's binned sums do not depend on how its waves were scheduled); the
// copies are zeroed for the next tile.  Callers wait at a barrier before
// the histograms are used again.
__device__ __forceinline__ void hist_flush(int nbins, int copies, double *hist, double *out,
                                           int tid, int nt)
{
    const int w = nbins + 1;
    for (int i = tid; i < w; i += nt) {
        double s = hist[i];
        hist[i] = 0.0;
        for (int c = 1; c < copies; ++c) {
            s += hist[c * w + i];
            hist[c * w + i] = 0.0;
        }
        out[i] = s;
    }
}

// The flush at the end of a binning block: as hist_flush, but slot nbins of
// the row gets the sum of all its slots (the zero mode included), bin 0
// first over 64 strided lanes and a fixed tree, so that the k-space Parseval
// sum is one more column of the reduction instead of a pass over its results.
__device__ __forceinline__ void hist_flush_row(int nbins, int copies, double *hist, double *out,
                                               int tid, int nt)
{
    const int w = nbins + 1;
    for (int i = tid; i < w; i += nt) {
        double s = hist[i];
        for (int c = 1; c < copies; ++c) s += hist[c * w + i];
        hist[i] = s;
        if (i < nbins) out[i] = s;
    }
    __syncthreads();
    if (tid < 64) {
        double t = 0.0;
        for (int i = tid; i < w; i += 64) t += hist[i];
        for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
        if (tid == 0) out[nbins] = t;
    }
}

// 1/d for d > 0 in FP64: the hardware reciprocal refined by one Newton step,
// which squares the estimate's relative error; the scale it feeds multiplies
// FP32 modes in FP64 and is rounded to FP32 with the product.
__device__ __forceinline__ double rcp_f64(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    return fma(fma(-d, r, 1.0), r, r);
}

// The thread index, hidden from the optimiser once per tile when OPAQUE: the
// per-thread LDS and global offsets derived from it are then recomputed in
// every tile instead of being hoisted out of the tile loop, where dozens of
// them would stay live (and spill) across the fused pass.  The empty asm
// statement emits no instruction.
template <bool OPAQUE>
__device__ __forceinline__ int opaque_tid(int tid)
{
    if constexpr (OPAQUE) asm volatile("" : "+v"(tid));
    return tid;
}

// ============================================================ strided tiles
// EPI = false: plain pass (no epilogue code, fewest registers);
// EPI = true : last-axis pass with the binning / Poisson epilogue.
// hist / edges: LDS arrays (EPI with binning only): a.hcopies histograms of
// nbins + 1 entries (wave w adds into copy w, or all into copy 0) and the
// edge table; the tile adds its w|F|^2 sums into them.
// K2 (EPI): 1 the continuous k^2 of the last axis from |n_z|, 2 its table,
// 0 either, chosen per call (fewer kernels, more registers).
// m^2 for 0 <= m < 2^12 (mode indices) with a full-rate 24-bit multiply.
__device__ __forceinline__ uint32_t sq24(int m) { return __umul24((unsigned)m, (unsigned)m); }

// Element offset of column f of a strided pass: outer group o = f / C,
// then f - o C within it.  Passes have fewer than 2^31 columns (at most
// (N0 / 2 + 1) N1 nc of a 2048^3 lattice), so 32-bit division suffices.
__device__ __forceinline__ int64_t col_base(const SArgs &a, int64_t f)
{
    const int fi = (int)f, c = (int)a.ncols_inner;
    const int o = fi / c;
    return (int64_t)o * a.outer + (fi - o * c);
}

template <int L, int S, bool EPI, int NT, bool NTM = false, int K2 = 0>
struct STile {
    static constexpr int B = s_b(L);
    static constexpr int RPT = NT / B;  // row groups in the epilogue
    static constexpr size_t O_BUF = 0, O_TW = al16(sizeof(c32) * L * B), BYTES = s_bytes(L);
    static __device__ void tables(const SArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, L, tid, NT);
    }
    // The fused tile's inputs: the first forward stage's inputs, rows
    // j + r L/R0 of the thread's column (radix R0), all loads issued before
    // any of them is used (a column past the end loads column 0 and is
    // zeroed).
    static constexpr RadixPlan PL = kPlan<L, kEpiPair>;  // of the fused pass
    static constexpr int R0 = PL.n == 0 ? 1 : PL.r[0];
    static constexpr int R01 = PL.n == 0 ? 1 : PL.r1[0];
    static constexpr int NB0 = col_nb(L, R0, B, NT);
    struct In {
        c32 v[NB0][R0];
    };
    static __device__ __forceinline__ void load_in(const SArgs &a, int64_t t, int tid, In &in)
    {
        constexpr int Q0 = L / R0;
        constexpr int JS = NT / B;
        const int col = tid % B;
        const int64_t f = t * B + col;
        const bool valid = f < a.ncols;
        // a column past the end reads column 0 (in bounds) and keeps zeros
        const int64_t base = valid ? col_base(a, f) : 0;
        const c32 *gin = (const c32 *)a.in + base;
        const int j0 = tid / B;
#pragma unroll
        for (int i = 0; i < NB0; ++i) {
            const int j = j0 + i * JS;
            if (Q0 % JS == 0 || j < Q0) {
                gload_pts<R0, NTM>(in.v[i], gin + (int64_t)j * a.stride, (int64_t)Q0 * a.stride,
                                   true);
#pragma unroll
                for (int r = 0; r < R0; ++r)
                    if (!valid) in.v[i][r] = c32{0.f, 0.f};
            } else {
#pragma unroll
                for (int r = 0; r < R0; ++r) in.v[i][r] = c32{0.f, 0.f};
            }
        }
    }

    // tab (EPI = false): the block's first tile, tables included.  Their
    // values are fetched first and go to LDS once the tile's own loads are
    // issued behind them, so that the two waits are one: a tile lives for
    // about 13 us, and a wait for the table ahead of its loads took 1 us of
    // them (512^3 real y 203 -> 187 us, 400^3 y 107 -> 99, 240 x 180 x 150
    // with three components z 36 -> 30, 128^3 y 9.4 -> 8.9; the y pass over
    // 256^3 complex, at 45.5 us near the rate its write-back allows, 47).
    static __device__ void tile(const SArgs &a, int64_t t, char *sm, int tid, double *hist,
                                const BinEdge *edges, bool tab = false)
    {
        if constexpr (EPI) {
            In in;
            load_in(a, t, tid, in);
            tile_in(a, t, sm, tid, hist, edges, in);
        } else if constexpr (S < 0 && table_first(L)) {
            if (tab) {
                tables(a, sm, tid);
                __syncthreads();
            }
            plain(a, t, sm, tid, NoHook{});
            __syncthreads();
        } else {
            TableRegs<L, NT> wt;
            if (tab) wt.load(a.tw, tid);
            plain(a, t, sm, tid, tab_hook([&] {
                if (!tab) return;
                wt.store((c32 *)(sm + O_TW), tid);
                if (kPaired<L>) __syncthreads();  // else the first stage reads no table
            }));
            __syncthreads();
        }
    }

    template <class Hook>
    static __device__ __forceinline__ void plain(const SArgs &a, int64_t t, char *sm, int tid,
                                                 Hook hook)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW);
        const int col = tid % B;
        const bool store = (a.epi & EPI_STORE) != 0;
        const int64_t f = t * B + col;
        const bool valid = f < a.ncols;
        const int64_t base = valid ? col_base(a, f) : 0;
        const c32 *gin = (const c32 *)a.in + base;
        c32 *gout = (c32 *)a.out + base;
        // global -> registers -> stages -> registers -> global
        col_fft<L, S, B, NT, true, true, 0, 1, NTM>(buf, gin, gout, a.stride, valid && store, tw,
                                                     tid, hook);
    }

    // The fused tile from its loaded inputs (load_in of the same t).
    static __device__ __forceinline__ void tile_in(const SArgs &a, int64_t t, char *sm, int tid,
                                                   double *hist, const BinEdge *edges, In &in)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW);
        const int col = tid % B;
        const int rg = tid / B;
        const bool store = (a.epi & EPI_STORE) != 0;
        const int64_t f = t * B + col;
        const bool valid = f < a.ncols;
        const int64_t base = valid ? col_base(a, f) : 0;
        c32 *gout = (c32 *)a.out + base;
        epilogue(a, buf, tw, tid, col, rg, f, valid, store, gout, hist, edges, in);
        __syncthreads();
    }

    // Last-axis epilogue.  The forward transform stops with its last stage in
    // registers: thread (col, j0) holds the modes kz = j + r QL of column col
    // for its butterflies j.  The Poisson scale is applied there, and the
    // backward transform runs its radices in reverse order, so that its first
    // stage (radix RL, inputs at points j + r QL) starts from those same
    // registers.  The P(k) sums need runs of consecutive kz (so that
    // neighbouring modes share a bin): for them the modes are also written
    // to LDS in natural order and thread (col, rg) walks kz in
    // [rg EP, rg EP + EP).
    static __device__ __forceinline__ void epilogue(const SArgs &a, c32 *buf, const c32 *tw,
                                                    int tid, int col, int rg, int64_t f,
                                                    bool valid, bool store, c32 *gout,
                                                    double *hist, const BinEdge *edges, In &in)
    {
        constexpr int NST = PL.n;
        constexpr int RL = NST == 0 ? 1 : PL.r[NST - 1];
        constexpr int RL1 = NST == 0 ? 1 : PL.r1[NST - 1];
        constexpr int QL = L / RL;
        constexpr int NB = col_nb(L, RL, B, NT);
        const int j0 = tid / B;
        // first forward stage (no twiddles) on the loaded inputs
#pragma unroll
        for (int i = 0; i < NB0; ++i) dft_first<L, R0, R01, S>(in.v[i], tw);
        c32 v[NB][RL];
        if constexpr (NST <= 1) {
            static_assert(NB0 == NB && R0 == RL, "one stage: its inputs are its butterflies");
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int r = 0; r < RL; ++r) v[i][r] = in.v[i][r];
        } else {
            col_stage_out<L, R0, 1, B, NT, false>(buf, nullptr, 0, false, tid, in.v);
            col_fft<L, S, B, NT, false, false, 1, R0, NTM, false, true, kEpiPair>(buf, nullptr, nullptr, 0,
                                                                      false, tw, tid);
            col_stage_in<L, RL, RL1, QL, S, B, NT, false>(buf, nullptr, 0, false, tw, tid, v);
        }
        // column f = ky nxk + kx of the (kx, ky) plane (fewer than 2^31 columns)
        const int kx = valid ? (int)f % a.mt.nxk : 0;
        const int ky = valid ? (int)f / a.mt.nxk : 0;
        const bool corner = kx == 0 && ky == 0;
        // the column's |n_x|, |n_y| (the r2c half spectrum holds kx <= N0 / 2)
        const int mx = 2 * kx <= a.mt.n0 ? kx : a.mt.n0 - kx;
        const int my = 2 * ky <= a.mt.n1 ? ky : a.mt.n1 - ky;
        // this wave's histogram
        double *wh = hist + (a.hcopies > 1 ? (tid >> 6) * (a.mt.nbins + 1) : 0);
        // q_x + q_y of the column (exact integers below 2^32)
        const uint32_t qxy = a.mt.qx_unit * sq24(mx) + a.mt.qy_unit * sq24(my);
        if (a.epi & EPI_PK) {
            col_stage_out<L, RL, QL, B, NT, false>(buf, nullptr, 0, false, tid, v);
            bin_walk(a, buf, col, rg, kx, corner, qxy, valid, wh, edges);
        }
        if (a.epi & EPI_POISSON) {
            if (K2 == 1 || (K2 == 0 && a.mt.k2z_unit > 0.0)) {
                // continuous k^2 from |n_x|, |n_y|, |n_z|
                const double k2xy = valid ? fma(a.mt.k2x_unit, (double)sq24(mx),
                                                a.mt.k2y_unit * (double)sq24(my))
                                          : 1.0;
                scale_modes<true>(a, v, j0, k2xy, corner);
            } else {
                // the tables
                const double k2xy = valid ? a.mt.k2[0][kx] + a.mt.k2[1][ky] : 1.0;
                scale_modes<false>(a, v, j0, k2xy, corner);
            }
        }
        if (a.epi & EPI_PK_AFTER) {
            col_stage_out<L, RL, QL, B, NT, false>(buf, nullptr, 0, false, tid, v);
            bin_walk(a, buf, col, rg, kx, corner, qxy, valid, wh, edges);
        }
        if constexpr (S < 0) {
            if (a.epi & EPI_POISSON) {
                // backward transform: first stage (radix RL, no twiddles) from
                // the registers, the rest through LDS in reverse radix order
#pragma unroll
                for (int i = 0; i < NB; ++i) dft_first<L, RL, RL1, +1>(v[i], tw);
                if constexpr (NST <= 1) {
                    col_stage_out<L, RL, 1, B, NT, true, NTM>(buf, gout, a.stride, valid && store,
                                                              tid, v);
                } else {
                    col_stage_out<L, RL, 1, B, NT, false>(buf, nullptr, 0, false, tid, v);
                    col_fft<L, +1, B, NT, false, true, 1, RL, NTM, true, false, kEpiPair>(
                        buf, nullptr, gout, a.stride, valid && store, tw, tid);
                }
                return;
            }
        }
        if (store)  // spectrum out: the modes are still in registers
            col_stage_out<L, RL, QL, B, NT, true, NTM>(buf, gout, a.stride, valid, tid, v);
    }

    // The Poisson scale -1/(N k^2) (FP64, rounded once with the product) of
    // the modes kz = j + r QL a thread holds after the forward transform.
    template <bool CONT, int RL, int NB>
    static __device__ __forceinline__ void scale_modes(const SArgs &a, c32 (&v)[NB][RL], int j0,
                                                       double k2xy, bool corner)
    {
        constexpr int QL = L / RL;
        constexpr int JS = NT / B;
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int j = j0 + i * JS;
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                const int kz = j + r * QL;
                if (QL % JS == 0 || j < QL) {
                    const int m = 2 * kz < L ? kz : L - kz;
                    const double k2z = CONT ? a.mt.k2z_unit * (double)sq24(m) : a.mt.k2[2][kz];
                    const double sc =
                        (corner && kz == 0) ? 0.0 : -a.mt.scale_n * rcp_f64(k2xy + k2z);
                    v[i][r] = c32{(float)((double)v[i][r].x * sc), (float)((double)v[i][r].y * sc)};
                }
            }
        }
    }

    // P(k) partial sums of the modes in LDS (natural order).  The modes kz
    // and L - kz have the same m = |n_z|, hence the same q and bin, so
    // thread (col, rg) walks m upward over its run [rg EH, rg EH + EH) of
    // 0 .. L/2 and takes both modes of each m (one at m = 0, and at m = L/2
    // for even L).  Along the run q = q_xy + m^2 q_u grows by integer
    // differences, and the bin changes where q reaches the current bin's
    // upper edge: to the next bin when one step of m never crosses two
    // thresholds (mt.walk1, checked when the thresholds are made), else to
    // the exact bin of q.  w |F|^2 sums go to `hist` -- the wave's own LDS
    // histogram, or the block's one -- at each change, in program order, so
    // with one histogram per wave the sums do not depend on scheduling.
    // Ends at a barrier, so LDS may be rewritten afterwards.
    static constexpr int MH = L / 2;                       // largest m
    static constexpr int EH = (MH + 1 + RPT - 1) / RPT;    // m values per row group
    static __device__ void bin_walk(const SArgs &a, const c32 *buf, int col, int rg, int kx,
                                    bool corner, uint32_t qxy, bool valid, double *hist,
                                    const BinEdge *edges)
    {
        const int nb = a.mt.nbins;
        const float cq = (float)((double)nb * nb / a.mt.qmax);
        // the half-spectrum weight is the same for the whole column
        const double wgt = (a.mt.half && !(kx == 0 || 2 * kx == a.mt.n0)) ? 2.0 : 1.0;
        const uint32_t qu = a.mt.qz_unit;
        const bool walk1 = a.mt.walk1 != 0;
        const int m0 = rg * EH;
        const int n = MH + 1 - m0 < EH ? MH + 1 - m0 : EH;  // may be <= 0
        if (valid && n > 0) {
            // q at m0 and its first difference (m0 + 1)^2 - m0^2 = 2 m0 + 1
            uint32_t q = qxy + sq24(m0) * qu;
            uint32_t dq = (uint32_t)(2 * m0 + 1) * qu;
            const uint32_t ddq = 2u * qu;
            // slot nbins: the zero mode (kept for the Parseval sum); q = 0
            // there, and the next mode's bin is then found from scratch
            int b;
            uint32_t hi;
            if (corner && m0 == 0) {
                b = nb;
                hi = 1u;
            } else {
                b = bin_edge(q, nb, cq, edges);
                hi = edges[b].hi;
            }
            double acc = 0.0;
#pragma unroll 4
            for (int e = 0; e < EH; ++e) {
                if (EH * RPT != MH + 1 && e >= n) break;
                const int m = m0 + e;
                const c32 u = buf[m * B + col];
                // the partner mode L - m (none for m = 0, the same mode for 2 m = L)
                const bool two = m != 0 && 2 * m != L;
                const c32 w = buf[(two ? L - m : m) * B + col];
                if (q >= hi) {
                    atomicAdd(&hist[b], wgt * acc);
                    acc = 0.0;
                    if (walk1 && b < nb)
                        ++b;
                    else
                        b = bin_edge(q, nb, cq, edges);
                    hi = edges[b].hi;
                }
                double pw = (double)u.x * u.x + (double)u.y * u.y;
                if (two) pw += (double)w.x * w.x + (double)w.y * w.y;
                acc += pw;
                q += dq;
                dq += ddq;
            }
            atomicAdd(&hist[b], wgt * acc);
        }
        __syncthreads();
    }
};

// Wide strided tile: twice the columns of STile (256-byte row segments at
// L = 512) with twice the threads, one block per CU: for long strides (the
// last axis of large or multi-component fields), where longer contiguous
// segments per row pay for the lower block count.  No epilogue.
constexpr int kSWThreads = 1024;

template <int L, int S, int NT, bool NTM = false>
struct STileW {
    static constexpr int B = 2 * s_b(L);
    static constexpr size_t O_BUF = 0, O_TW = al16(sizeof(c32) * L * B),
                            BYTES = al16(O_TW + sizeof(c32) * L);
    static __device__ void tables(const SArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, L, tid, NT);
    }
    static __device__ void tile(const SArgs &a, int64_t t, char *sm, int tid)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW);
        const int col = tid % B;
        const int64_t f = t * B + col;
        const bool valid = f < a.ncols;
        const int64_t base = valid ? col_base(a, f) : 0;
        col_fft<L, S, B, NT, true, true, 0, 1, NTM>(buf, (const c32 *)a.in + base, (c32 *)a.out + base,
                                         a.stride, valid && (a.epi & EPI_STORE) != 0, tw, tid);
        __syncthreads();
    }
};

// Transposing strided tile for the z pass of a c2c plan in the paper's
// k-space order (k_z, k_x, k_y): every column's points are contiguous there
// (stride ncomp).  Forward (EPI_TSTORE): natural columns in, the last stage
// writes LDS and the tile is stored point-fastest; backward (EPI_TLOAD): the
// tile is loaded point-fastest into LDS and the last stage writes the
// natural columns.  Threads walk the tile's (column, point) pairs with the
// point fastest, so each column's run is read or written contiguously.
template <int L, int S, int NT>
struct STileT {
    static constexpr int B = s_b(L);
    static constexpr size_t O_BUF = 0, O_TW = al16(sizeof(c32) * L * B),
                            BYTES = al16(O_TW + sizeof(c32) * L);
    static __device__ void tables(const SArgs &a, char *sm, int tid)
    {
        load_table((c32 *)(sm + O_TW), a.tw, L, tid, NT);
    }
    static __device__ __forceinline__ int64_t tpos(const SArgs &a, int64_t f, int kz)
    {
        const int64_t c1 = a.t_n0 * a.t_nc;
        const int64_t y = f / c1, r = f - y * c1;
        const int64_t x = r / a.t_nc, c = r - x * a.t_nc;
        return ((y * a.t_n0 + x) * a.t_n2 + kz) * a.t_nc + c;
    }
    static __device__ void tile(const SArgs &a, int64_t t, char *sm, int tid)
    {
        c32 *buf = (c32 *)(sm + O_BUF);
        const c32 *tw = (const c32 *)(sm + O_TW);
        const int col = tid % B;
        const int64_t f0 = t * B;
        const int64_t f = f0 + col;
        const bool valid = f < a.ncols;
        const int64_t base = valid ? f : 0;  // natural z pass: column f at f
        if (a.epi & EPI_TLOAD) {
            const c32 *in = (const c32 *)a.in;
            for (int e = tid; e < B * L; e += NT) {
                const int kz = e % L, cl = e / L;
                const int64_t ff = f0 + cl;
                buf[kz * B + cl] = ff < a.ncols ? in[tpos(a, ff, kz)] : c32{0.f, 0.f};
            }
            __syncthreads();
            col_fft<L, S, B, NT, false, true>(buf, nullptr, (c32 *)a.out + base, a.stride, valid,
                                              tw, tid);
        } else {
            col_fft<L, S, B, NT, true, false>(buf, (const c32 *)a.in + base, nullptr, a.stride,
                                              valid, tw, tid);
            c32 *out = (c32 *)a.out;
            for (int e = tid; e < B * L; e += NT) {
                const int kz = e % L, cl = e / L;
                const int64_t ff = f0 + cl;
                if (ff < a.ncols) out[tpos(a, ff, kz)] = buf[kz * B + cl];
            }
        }
        __syncthreads();
    }
};

// ======================================================= standalone kernels
// One x tile per block (tile index = blockIdx.x).

template <int M, int NC>
__global__ __launch_bounds__(kXThreads) void k_x_r2c(XArgs a)
{
    using T = XR2CGen<M, NC, kXThreads>;
    __shared__ __align__(16) char sm[T::BYTES];
    T::tile(a, blockIdx.x, sm, threadIdx.x, a.sumsq ? a.sumsq + blockIdx.x : nullptr, true);
}

template <int M, int NC>
__global__ __launch_bounds__(kXThreads) void k_x_c2r(XArgs a)
{
    using T = XC2RGen<M, NC, kXThreads>;
    __shared__ __align__(16) char sm[T::BYTES];
    T::tile(a, blockIdx.x, sm, threadIdx.x, true);
}

template <int M>
__global__ __launch_bounds__(kXThreads) void k_x_r2c_v(XArgs a)
{
    using T = XR2CV<M, kXThreads>;
    __shared__ __align__(16) char sm[T::BYTES];
    T::tile(a, blockIdx.x, sm, threadIdx.x, a.sumsq ? a.sumsq + blockIdx.x : nullptr, true);
}

template <int M>
__global__ __launch_bounds__(kXThreads) void k_x_c2r_v(XArgs a)
{
    using T = XC2RV<M, kXThreads>;
    __shared__ __align__(16) char sm[T::BYTES];
    T::tile(a, blockIdx.x, sm, threadIdx.x, true);
}

template <int L, int NC, int S>
__global__ __launch_bounds__(kXThreads) void k_x_c2c_v(XArgs a)
{
    using T = XC2CV<L, NC, S, kXThreads>;
    __shared__ __align__(16) char sm[T::BYTES];
    T::tile(a, blockIdx.x, sm, threadIdx.x, true);
}

// The XCD-aware walk of the strided passes over virtual block ids
// vb = blockIdx.x + i * G (G is a multiple of 8).  The chip hands block ids to
// its 8 XCDs in turn, so vb mod 8 is this block's XCD.  Chunks of K
// consecutive tiles go to one XCD and the chunks rotate over the XCDs:
// neighbouring tiles, which share cache lines when rows are not 128-byte
// aligned, meet in one L2, while all XCDs stream from nearby addresses.
// Passes have fewer than 2^31 columns, so tiles and ids are 32-bit.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t vb, uint32_t K)
{
    const uint32_t lb = vb / 8, c = lb / K;
    return (c * 8 + (vb % 8)) * K + (lb - c * K);
}

// Strided pass: persistent-style walk over tiles where they are binned.
// Occupancy target: four waves per SIMD (two blocks per CU) except where the
// fused pass's LDS tables leave room for one block (lines of 1024 points and
// more), where two waves per SIMD are all it can reach.
template <int L, int S, bool EPI, bool NTM = false, int K2 = 0>
__global__ __launch_bounds__(EPI ? e_nt<L> : s_nt<L>)
    __attribute__((amdgpu_waves_per_eu(EPI && L >= 1024 ? 2 : 4))) void k_strided(SArgs a)
{
    constexpr int NT = EPI ? e_nt<L> : s_nt<L>;
    using T = STile<L, S, EPI, NT, NTM, K2>;
    constexpr int B = T::B;
    __shared__ __align__(16) char sm[T::BYTES];
    extern __shared__ double dyn[];  // hist[hcopies][nbins + 1], edges[nbins + 1]
    const int tid = threadIdx.x;
    const uint32_t ntiles = (uint32_t)((a.ncols + B - 1) / B), K = a.xcd_chunk;
    if constexpr (!EPI) {
        // one tile a block (s_grid)
        const uint32_t t = xcd_tile(blockIdx.x, K);
        if (t < ntiles) T::tile(a, t, sm, tid, nullptr, nullptr, true);
        return;
    }
    T::tables(a, sm, tid);
    const bool pk = EPI && (a.epi & (EPI_PK | EPI_PK_AFTER)) != 0;
    const int nb = a.mt.nbins;
    double *hist = dyn;
    BinEdge *edges = (BinEdge *)(dyn + a.hcopies * (nb + 1));
    if (pk) hist_init(a.mt, a.hcopies, hist, edges, tid, NT);
    __syncthreads();
    const uint32_t span = (ntiles + 8 * K - 1) / (8 * K) * (8 * K);
    for (uint32_t vb = blockIdx.x; vb < span; vb += gridDim.x) {
        const uint32_t t = xcd_tile(vb, K);
        if (t >= ntiles) continue;  // uniform over the block
        T::tile(a, t, sm, opaque_tid<EPI>(tid), hist, edges);
    }
    if (pk) {
        __syncthreads();
        hist_flush_row(nb, a.hcopies, hist, a.partial + (int64_t)blockIdx.x * (nb + 1), tid, NT);
    }
}

template <int L, int S, bool NTM = false>
__global__ __launch_bounds__(kSWThreads) void k_strided_w(SArgs a)
{
    using T = STileW<L, S, kSWThreads, NTM>;
    constexpr int B = T::B;
    __shared__ __align__(16) char sm[T::BYTES];
    const int tid = threadIdx.x;
    T::tables(a, sm, tid);
    __syncthreads();
    const uint32_t ntiles = (uint32_t)((a.ncols + B - 1) / B), K = a.xcd_chunk;
    const uint32_t span = (ntiles + 8 * K - 1) / (8 * K) * (8 * K);
    for (uint32_t vb = blockIdx.x; vb < span; vb += gridDim.x) {
        const uint32_t t = xcd_tile(vb, K);
        if (t >= ntiles) continue;  // uniform over the block
        T::tile(a, t, sm, tid);
    }
}

template <int L, int S>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_strided_t(SArgs a)
{
    using T = STileT<L, S, kSThreads>;
    __shared__ __align__(16) char sm[T::BYTES];
    const int tid = threadIdx.x;
    T::tables(a, sm, tid);
    __syncthreads();
    const int64_t ntiles = (a.ncols + T::B - 1) / T::B;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) T::tile(a, t, sm, tid);
}

// Grid of a narrow strided pass: every tile of the walk a block (the plain
// pass), at most grid_cap blocks (the fused one), at most a round of them
// where they bin.
template <int L>
inline int s_grid(const SArgs &a, int grid_cap, size_t shm)
{
    const int64_t chunk = a.xcd_chunk, ntiles = (a.ncols + s_b(L) - 1) / s_b(L);
    const int64_t span = (ntiles + 8 * chunk - 1) / (8 * chunk) * (8 * chunk);
    if ((a.epi & (EPI_PK | EPI_PK_AFTER | EPI_POISSON)) == 0) return (int)span;
    if (a.epi & (EPI_PK | EPI_PK_AFTER))
        grid_cap = binning_blocks(L, grid_cap, s_bytes(L) + shm, e_nt<L> / 64);
    return (int)(span < grid_cap ? span : grid_cap);
}

}  // namespace lf2
