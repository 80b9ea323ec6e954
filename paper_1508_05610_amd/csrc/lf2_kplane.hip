// lf2_kplane.hip -- the x and y transforms of one z plane in one block: for
// small lattices whose planes fit a block's LDS twice, one launch and one
// pass over memory in place of two.
//
// Such lattices are bound by launches and latency, not by bytes: a 32^3
// r2c transform moves 0.4 MB, and its x and y passes took 5.9 and 3.2 us on
// the device and about 3 us of host time per launch.  The first stage of the
// first axis takes its points from memory, the last stage of the other
// stores them; between them every stage reads one LDS buffer and writes the
// other, the split and the merge of the half-length real transform read as
// part of the stage after them.  An r2c or c2r direction of a 16^3 to 96^3
// lattice: 13.2-22.7 us in two passes, 10.3-18.5 us here (the z pass
// included); Poisson with 32 bins at 32^3 29 -> 23 us, at 64^3 35 -> 28 us,
// at 108^3 60 -> 51 us.
//
// The line lengths are run-time arguments (one kernel per transform kind
// instead of one per pair of lengths): each stage's divisions are by magic
// numbers the host prepares, and the radices are the compiled kernels'
// factors in their order.  A thread holds one butterfly at a time.
#include "lf2_kernels.hpp"

namespace lf2 {

// n / d for n < 2^16 by a multiply (m = ceil(2^32 / d)): the error of m is
// below d, so n (m d - 2^32) < 2^32 whenever n d < 2^32.
struct PDiv {
    uint32_t d, m;  // m = 0: d = 1
    __device__ __forceinline__ int div(int n) const { return m ? (int)__umulhi((uint32_t)n, m) : n; }
};

struct PStage {
    int r, ns, q, tstep;  // radix, points combined before, L / r, L / (ns r)
    PDiv dq, dns;         // by q (x lines) and by ns
};

struct PAxis {
    int len, n, ragged;   // ragged: a line of the run-time schedules (kPaired)
    PStage st[kPlaneStages];
    const void *tw;
};

struct PlaneArgs {
    XArgs x;              // offsets and strides of both sides, twiddles, sumsq
    int nc, n1, lp, np;   // components, rows of a plane, LDS line pitch, points of a k-space row
    PDiv dcol, dnc;       // by np nc and by nc
    PAxis ax, ay;
};

// Where a stage's butterflies take their points from and leave them.
enum : int {
    P_LDS = 0,   // the LDS lines
    P_MEM = 1,   // the plane in memory
    P_HALF = 2   // the LDS lines, through the half-length real transform's
                 // split (y forward) or merge (x backward) of bins k, M - k
};

struct PBlock {
    c32 *src, *dst;             // LDS lines
    const void *in;             // the plane in memory
    void *out;
    const c32 *twx, *twy, *twp;
    int tid, nt;
    double ss;                  // this thread's sum of squares of a real input
};

// XW: twiddle_mul's; the stage's radix-R butterfly on v.
template <int R, int S>
__device__ __forceinline__ void pbutterfly(c32 (&v)[R], const PStage &st, int k, const c32 *tw,
                                           bool xw)
{
    if (st.ns > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) {
            c32 w = tw[__umul24(r * k, st.tstep)];
            if (S > 0) w = conjg(w);
            v[r] = xw ? twiddle_mul<true>(v[r], w) : twiddle_mul(v[r], w);
        }
    }
    dft_fixed<R, S, true>(v);
}

// One stage on lines along x: line l = y nc + i at l lp, points padded;
// consecutive threads take consecutive butterflies of a line.  REAL: the
// plane in memory holds real rows (pairs of floats), else complex ones.
template <int R, int S, int SRC, int DST, bool REAL>
__device__ __forceinline__ void stage_x(const PlaneArgs &a, const PStage &st, PBlock &p, bool xw)
{
    const int nc = a.nc, M = a.ax.len;
    for (int b = p.tid; b < a.n1 * nc * st.q; b += p.nt) {
        const int l = st.dq.div(b), j = b - l * st.q;
        const int kb = st.dns.div(j), k = j - kb * st.ns;
        const c32 *line = p.src + l * a.lp;
        c32 v[R];
        if (SRC == P_MEM) {
            const int y = nc == 1 ? l : a.dnc.div(l), i = l - y * nc;
            if (REAL) {
                // point n is the pair of floats (2n) nc + i, (2n + 1) nc + i
                const float *row = (const float *)p.in + (int64_t)y * a.x.in_row + i;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float *f = row + 2 * (j + r * st.q) * nc;
                    v[r] = c32{f[0], f[nc]};
                }
                if (a.x.sumsq) {
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        p.ss += (double)v[r].x * v[r].x + (double)v[r].y * v[r].y;
                }
            } else {
                const c32 *row = (const c32 *)p.in + (int64_t)y * a.x.in_row + i;
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = row[(j + r * st.q) * nc];
            }
        } else if (SRC == P_HALF) {
            // Z[n] = (X[n] + conj X[M-n]) + i W^{-n} (X[n] - conj X[M-n])
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int n = j + r * st.q;
                c32 xk = line[lpad(n)], xm = line[lpad(M - n)];
                if (n == 0) {
                    xk.y = 0.f;
                    xm.y = 0.f;
                }
                const c32 s1 = add(xk, conjg(xm));
                const c32 d1 = mul(conjg(p.twp[n]), sub(xk, conjg(xm)));
                v[r] = c32{s1.x - d1.y, s1.y + d1.x};
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = line[lpad(j + r * st.q)];
        }
        pbutterfly<R, S>(v, st, k, p.twx, xw);
        const int p0 = kb * st.ns * R + k;
        if (DST == P_MEM) {
            const int y = nc == 1 ? l : a.dnc.div(l), i = l - y * nc;
            if (REAL) {
                float *row = (float *)p.out + (int64_t)y * a.x.out_row + i;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float *f = row + 2 * (p0 + r * st.ns) * nc;
                    f[0] = v[r].x;
                    f[nc] = v[r].y;
                }
            } else {
                c32 *row = (c32 *)p.out + (int64_t)y * a.x.out_row + i;
#pragma unroll
                for (int r = 0; r < R; ++r) row[(p0 + r * st.ns) * nc] = v[r];
            }
        } else {
            c32 *out = p.dst + l * a.lp;
#pragma unroll
            for (int r = 0; r < R; ++r) out[lpad(p0 + r * st.ns)] = v[r];
        }
    }
}

// One stage on columns along y: column (c, i) of point c and component i at
// i lp + lpad(c), rows nc lp apart; consecutive threads take consecutive
// elements of a k-space row.
template <int R, int S, int SRC, int DST>
__device__ __forceinline__ void stage_y(const PlaneArgs &a, const PStage &st, PBlock &p, bool xw)
{
    const int nc = a.nc, M = a.ax.len, ncol = a.np * nc, rs = nc * a.lp;
    for (int b = p.tid; b < ncol * st.q; b += p.nt) {
        const int j = a.dcol.div(b), q = b - j * ncol;
        const int kb = st.dns.div(j), k = j - kb * st.ns;
        const int c = nc == 1 ? q : a.dnc.div(q), i = q - c * nc;
        const int at = i * a.lp + lpad(c);
        c32 v[R];
        if (SRC == P_MEM) {
            const c32 *in = (const c32 *)p.in + q;
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = in[(int64_t)(j + r * st.q) * a.x.in_row];
        } else if (SRC == P_HALF) {
            // X[c] = fe + W^c fo, fe = (Z[c] + conj Z[M-c]) / 2,
            // fo = (Z[c] - conj Z[M-c]) / (2i), indices mod M
            const int c0 = c == M ? 0 : c, c1 = c == 0 || c == M ? 0 : M - c;
            const c32 w = p.twp[c];
            const c32 *base = p.src + i * a.lp;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const c32 *line = base + (j + r * st.q) * rs;
                const c32 z = line[lpad(c0)], zc = conjg(line[lpad(c1)]);
                const c32 fe = scl(add(z, zc), 0.5f);
                const c32 d = sub(z, zc);
                v[r] = add(fe, mul(w, c32{0.5f * d.y, -0.5f * d.x}));
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = p.src[at + (j + r * st.q) * rs];
        }
        pbutterfly<R, S>(v, st, k, p.twy, xw);
        const int p0 = kb * st.ns * R + k;
        if (DST == P_MEM) {
            c32 *o = (c32 *)p.out + q + (int64_t)p0 * a.x.out_row;
#pragma unroll
            for (int r = 0; r < R; ++r) o[(int64_t)(r * st.ns) * a.x.out_row] = v[r];
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) p.dst[at + (p0 + r * st.ns) * rs] = v[r];
        }
    }
}

#define LF2_RADIX(R_, CALL)  \
    switch (R_) {            \
    case 2: CALL(2); break;  \
    case 3: CALL(3); break;  \
    case 4: CALL(4); break;  \
    case 5: CALL(5); break;  \
    case 8: CALL(8); break;  \
    default: CALL(16); break; \
    }

__device__ __forceinline__ void pswap(PBlock &p)
{
    __syncthreads();
    c32 *t = p.src;
    p.src = p.dst;
    p.dst = t;
}

// All stages of an axis: the first from SRC, the last to DST (the others, and
// the lines between the axes, in LDS).
template <int S, int SRC, int DST, bool REAL>
__device__ void axis_x(const PlaneArgs &a, PBlock &p, bool xw_last)
{
    const int n = a.ax.n;
    for (int s = 0; s < n; ++s) {
        const PStage &st = a.ax.st[s];
        const bool first = s == 0, last = s == n - 1;
        const bool xw = last && xw_last && !a.ax.ragged;
        if (SRC != P_LDS && first && DST != P_LDS && last) {
#define CALL(R) stage_x<R, S, SRC, DST, REAL>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        } else if (SRC != P_LDS && first) {
#define CALL(R) stage_x<R, S, SRC, P_LDS, REAL>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        } else if (DST != P_LDS && last) {
#define CALL(R) stage_x<R, S, P_LDS, DST, REAL>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        } else {
#define CALL(R) stage_x<R, S, P_LDS, P_LDS, REAL>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        }
        if (!(DST != P_LDS && last)) pswap(p);
    }
}

template <int S, int SRC, int DST>
__device__ void axis_y(const PlaneArgs &a, PBlock &p)
{
    const int n = a.ay.n;
    for (int s = 0; s < n; ++s) {
        const PStage &st = a.ay.st[s];
        const bool first = s == 0, last = s == n - 1;
        const bool xw = last && !a.ay.ragged;
        if (SRC != P_LDS && first && DST != P_LDS && last) {
#define CALL(R) stage_y<R, S, SRC, DST>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        } else if (SRC != P_LDS && first) {
#define CALL(R) stage_y<R, S, SRC, P_LDS>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        } else if (DST != P_LDS && last) {
#define CALL(R) stage_y<R, S, P_LDS, DST>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        } else {
#define CALL(R) stage_y<R, S, P_LDS, P_LDS>(a, st, p, xw)
            LF2_RADIX(st.r, CALL)
#undef CALL
        }
        if (!(DST != P_LDS && last)) pswap(p);
    }
}

// LDS: two buffers of the plane's lines, the three twiddle tables, the block
// sum.
size_t plane_lds_bytes(int m, int np, int nc, int n1)
{
    return 8 * (2 * (size_t)row_pitch(np) * nc * n1 + (size_t)m + n1 + np) + 8 * 16;
}

// MODE 0: c2c, x then y for S < 0 and y then x for S > 0; 1: r2c x, y
// forward; 2: y backward, c2r x.  One block per plane.
template <int MODE, int S>
__global__ __launch_bounds__(1024) void k_plane(PlaneArgs a)
{
    extern __shared__ __align__(16) char psm[];
    const int M = a.ax.len, np = a.np, nlines = a.n1 * a.nc;
    PBlock p;
    p.tid = threadIdx.x;
    p.nt = blockDim.x;
    p.src = (c32 *)psm;
    p.dst = p.src + nlines * a.lp;
    c32 *twx = p.dst + nlines * a.lp, *twy = twx + M, *twp = twy + a.n1;
    double *red = (double *)(twp + np);
    p.twx = twx;
    p.twy = twy;
    p.twp = twp;
    p.ss = 0.0;
    const int64_t ib = a.x.in_off + (int64_t)blockIdx.x * a.x.in_plane;
    const int64_t ob = a.x.out_off + (int64_t)blockIdx.x * a.x.out_plane;
    p.in = MODE == 1 ? (const void *)((const float *)a.x.in + ib) : (const void *)((const c32 *)a.x.in + ib);
    p.out = MODE == 2 ? (void *)((float *)a.x.out + ob) : (void *)((c32 *)a.x.out + ob);
    // the first stages read no twiddles; their end barrier covers the tables
    for (int i = p.tid; i < M; i += p.nt) twx[i] = ((const c32 *)a.ax.tw)[i];
    for (int i = p.tid; i < a.n1; i += p.nt) twy[i] = ((const c32 *)a.ay.tw)[i];
    if (MODE != 0)
        for (int i = p.tid; i < np; i += p.nt) twp[i] = ((const c32 *)a.x.tw_post)[i];
    if constexpr (MODE == 1) {
        axis_x<S, P_MEM, P_LDS, true>(a, p, false);
        if (a.x.sumsq) {
            double ss = p.ss;
            for (int off = 32; off > 0; off >>= 1) ss += __shfl_down(ss, off, 64);
            if ((p.tid & 63) == 0) red[p.tid >> 6] = ss;
            __syncthreads();
            if (p.tid == 0) {
                double t = 0;
                for (int w = 0; w < p.nt / 64; ++w) t += red[w];
                a.x.sumsq[blockIdx.x] = t;
            }
        }
        axis_y<S, P_HALF, P_MEM>(a, p);
    } else if constexpr (MODE == 2) {
        axis_y<S, P_MEM, P_LDS>(a, p);
        axis_x<S, P_HALF, P_MEM, true>(a, p, false);
    } else if constexpr (S < 0) {
        axis_x<S, P_MEM, P_LDS, false>(a, p, true);
        axis_y<S, P_LDS, P_MEM>(a, p);
    } else {
        axis_y<S, P_MEM, P_LDS>(a, p);
        axis_x<S, P_LDS, P_MEM, false>(a, p, true);
    }
}

static PDiv pdiv(int d)
{
    return PDiv{(uint32_t)d, d == 1 ? 0u : (uint32_t)(((uint64_t)1 << 32) / d + (((uint64_t)1 << 32) % d ? 1 : 0))};
}

// The factors of a line as stages.
static void plane_axis(int len, const void *tw, PAxis &a)
{
    const RadixPlan p = radix_plan(len);
    a.len = len;
    a.n = p.nf;
    a.ragged = p.nodd > 1;
    a.tw = tw;
    int ns = 1;
    for (int i = 0; i < p.nf; ++i) {
        PStage &s = a.st[i];
        s.r = p.f[i];
        s.ns = ns;
        s.q = len / s.r;
        s.tstep = len / (ns * s.r);
        s.dq = pdiv(s.q);
        s.dns = pdiv(ns);
        ns *= s.r;
    }
}

// (Lines with a factor of 16 beside several of 3 and 5 would need the other
// rounding of the 16-point butterfly; they are 144 points and longer.)
bool plane_axis_ok(int len)
{
    const RadixPlan p = radix_plan(len);
    return len > 1 && p.nf <= kPlaneStages && !(p.nodd > 1 && p.f[0] == 16);
}

// Forward, a stage rounds as the two passes' stage does (twiddle_mul,
// dft_fixed) except where the compiler chose otherwise there: on
// run-time-schedule lines always; on compiled ones not the 16-point
// butterfly (real x lines of 16 points excepted) nor, on y and complex x
// lines, the 5-point one; not on y lines of three power-of-two stages (512
// points: 8, 8, 8), where P(k) moved by 1e-9 to 6e-9; and not on compiled
// complex x lines of two stages and more, whose last twiddles it rounds one way
// in some of a thread's butterflies and another way in others.
bool plane_axis_bits(int len, PlaneAxis axis)
{
    const RadixPlan p = radix_plan(len);
    if (p.nodd > 1) return true;
    const bool f16 = p.f[0] == 16, f5 = p.f[p.nf - 1] == 5;
    if (axis == PLANE_X_REAL) return !f16 || len == 16;
    const bool f222 = p.nodd == 0 && p.nf > 2;
    return !f16 && !f5 && (axis == PLANE_Y ? !f222 : p.nf == 1);
}

hipError_t launch_plane(int mode, int sign, const XArgs &x, int m, int np, int nc, int n1, int n2,
                        const void *tw_y, hipStream_t s)
{
    const size_t shm = plane_lds_bytes(m, np, nc, n1);
    if (!plane_axis_ok(m) || !plane_axis_ok(n1) || shm > 160 * 1024 || n2 < 1)
        return hipErrorInvalidValue;
    PlaneArgs a{};
    a.x = x;
    a.nc = nc;
    a.n1 = n1;
    a.np = np;
    a.lp = row_pitch(np);
    a.dcol = pdiv(np * nc);
    a.dnc = pdiv(nc);
    plane_axis(m, x.tw, a.ax);
    plane_axis(n1, tw_y, a.ay);
    // Whole waves of about four values a thread while every plane can have a
    // CU to itself (latency counts: 64^3 forward 12.7 us, 13.0 with eight and
    // 14.7 with sixteen), eight past that, where blocks share CUs (64 x 64 x
    // 1024 forward 32 us, 38 with four and 33 with sixteen).
    int nt = (n1 * nc * np / (n2 <= 256 ? 4 : 8) + 63) / 64 * 64;
    nt = nt < 128 ? 128 : nt > 1024 ? 1024 : nt;
    const dim3 g((unsigned)n2), t((unsigned)nt);
    if (mode == 1)
        hipLaunchKernelGGL((k_plane<1, -1>), g, t, shm, s, a);
    else if (mode == 2)
        hipLaunchKernelGGL((k_plane<2, 1>), g, t, shm, s, a);
    else if (sign < 0)
        hipLaunchKernelGGL((k_plane<0, -1>), g, t, shm, s, a);
    else
        hipLaunchKernelGGL((k_plane<0, 1>), g, t, shm, s, a);
    return hipGetLastError();
}

}  // namespace lf2
