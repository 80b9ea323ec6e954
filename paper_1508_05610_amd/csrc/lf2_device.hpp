// lf2_device.hpp -- device-side FFT engine for gfx950.
//
// Radix butterflies and an LDS-resident Stockham (autosort, decimation in
// time) driver.  One stage of radix R on a line of length L, after the
// stages already done have combined sub-transforms of length Ns, computes
// for every butterfly j in [0, L/R):
//   v_r = a[j + r L/R] * W_{Ns R}^{S r (j mod Ns)}        (r = 0..R-1)
//   v   = DFT_R(v)
//   b[(j div Ns) Ns R + (j mod Ns) + r Ns] = v_r
// and after the last stage the line holds its DFT in natural order.  Any
// order of radices whose product is L works; W_n = exp(2 pi i / n), S = -1
// forward and +1 backward.
//
// Lines live in LDS at address  line * LS + point * PS  (LS/PS chosen by the
// caller: contiguous lines for the x pass, interleaved columns for the
// strided passes so that lanes touch consecutive words).  A stage first
// reads every butterfly input of the thread into registers, waits at a
// barrier, then writes its outputs in place, and waits again.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lf2 {

struct c32 {
    float x, y;
};

__device__ __forceinline__ c32 mk(float a, float b) { return c32{a, b}; }
__device__ __forceinline__ c32 add(c32 a, c32 b) { return c32{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ c32 sub(c32 a, c32 b) { return c32{a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ c32 mul(c32 a, c32 b)
{
    return c32{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
__device__ __forceinline__ c32 conjg(c32 a) { return c32{a.x, -a.y}; }
__device__ __forceinline__ c32 scl(c32 a, float s) { return c32{a.x * s, a.y * s}; }
// s * i * a  (s = +-1)
template <int S>
__device__ __forceinline__ c32 muli(c32 a)
{
    return S > 0 ? c32{-a.y, a.x} : c32{a.y, -a.x};
}

// ---------------------------------------------------------------- butterflies
// In-place DFT of R values: v_k <- sum_r v_r exp(S 2 pi i r k / R).

template <int R, int S>
struct Dft;

template <int S>
struct Dft<1, S> {
    static __device__ __forceinline__ void run(c32 *) {}
};

template <int S>
struct Dft<2, S> {
    static __device__ __forceinline__ void run(c32 *v)
    {
        c32 a = v[0], b = v[1];
        v[0] = add(a, b);
        v[1] = sub(a, b);
    }
};

template <int S>
struct Dft<3, S> {
    static __device__ __forceinline__ void run(c32 *v)
    {
        const float h = 0.86602540378443864676f;  // sin(2 pi / 3)
        c32 t = add(v[1], v[2]);
        c32 u = sub(v[1], v[2]);
        c32 m = c32{v[0].x - 0.5f * t.x, v[0].y - 0.5f * t.y};
        c32 r = muli<S>(scl(u, h));
        v[0] = add(v[0], t);
        v[1] = add(m, r);
        v[2] = sub(m, r);
    }
};

template <int S>
struct Dft<4, S> {
    static __device__ __forceinline__ void run(c32 *v)
    {
        c32 a = add(v[0], v[2]), b = sub(v[0], v[2]);
        c32 c = add(v[1], v[3]), d = muli<S>(sub(v[1], v[3]));
        v[0] = add(a, c);
        v[2] = sub(a, c);
        v[1] = add(b, d);
        v[3] = sub(b, d);
    }
};

template <int S>
struct Dft<5, S> {
    static __device__ __forceinline__ void run(c32 *v)
    {
        const float c1 = 0.30901699437494742410f;   // cos(2 pi / 5)
        const float c2 = -0.80901699437494742410f;  // cos(4 pi / 5)
        const float s1 = 0.95105651629515357212f;   // sin(2 pi / 5)
        const float s2 = 0.58778525229247312917f;   // sin(4 pi / 5)
        c32 t1 = add(v[1], v[4]), t2 = add(v[2], v[3]);
        c32 t3 = sub(v[1], v[4]), t4 = sub(v[2], v[3]);
        c32 a0 = v[0];
        c32 m1 = c32{a0.x + c1 * t1.x + c2 * t2.x, a0.y + c1 * t1.y + c2 * t2.y};
        c32 m2 = c32{a0.x + c2 * t1.x + c1 * t2.x, a0.y + c2 * t1.y + c1 * t2.y};
        c32 n1 = muli<S>(c32{s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y});
        c32 n2 = muli<S>(c32{s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y});
        v[0] = add(a0, add(t1, t2));
        v[1] = add(m1, n1);
        v[4] = sub(m1, n1);
        v[2] = add(m2, n2);
        v[3] = sub(m2, n2);
    }
};

template <int S>
struct Dft<8, S> {
    static __device__ __forceinline__ void run(c32 *v)
    {
        const float r2 = 0.70710678118654752440f;
        c32 e[4] = {v[0], v[2], v[4], v[6]};
        c32 o[4] = {v[1], v[3], v[5], v[7]};
        Dft<4, S>::run(e);
        Dft<4, S>::run(o);
        // o[k] *= W8^{S k}
        o[1] = c32{r2 * (o[1].x - S * o[1].y), r2 * (o[1].y + S * o[1].x)};
        o[2] = muli<S>(o[2]);
        o[3] = c32{r2 * (-o[3].x - S * o[3].y), r2 * (-o[3].y + S * o[3].x)};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = add(e[k], o[k]);
            v[k + 4] = sub(e[k], o[k]);
        }
    }
};

template <int S>
struct Dft<16, S> {
    static __device__ __forceinline__ void run(c32 *v)
    {
        // 4 x 4: inner DFT4 over n1 (stride 4), twiddle W16^{n2 k1}, outer DFT4 over n2.
        const float c1 = 0.92387953251128675613f;  // cos(pi/8)
        const float s1 = 0.38268343236508977173f;  // sin(pi/8)
        const float r2 = 0.70710678118654752440f;
        c32 t[4][4];
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) {
#pragma unroll
            for (int n1 = 0; n1 < 4; ++n1) t[n2][n1] = v[4 * n1 + n2];
            Dft<4, S>::run(t[n2]);
        }
        // twiddles W16^{S n2 k1}: angle = S 2 pi n2 k1 / 16
        // n2 = 1: k1 = 1,2,3 -> (c1, S s1), (r2, S r2), (s1, S c1)
        // n2 = 2: k1 = 1,2,3 -> (r2, S r2), (0, S), (-r2, S r2)
        // n2 = 3: k1 = 1,2,3 -> (s1, S c1), (-r2, S r2), (-c1, -S s1)
        const c32 w11 = c32{c1, S * s1}, w12 = c32{r2, S * r2}, w13 = c32{s1, S * c1};
        const c32 w22 = c32{0.f, (float)S}, w23 = c32{-r2, S * r2};
        const c32 w33 = c32{-c1, -S * s1};
        t[1][1] = mul(t[1][1], w11);
        t[1][2] = mul(t[1][2], w12);
        t[1][3] = mul(t[1][3], w13);
        t[2][1] = mul(t[2][1], w12);
        t[2][2] = mul(t[2][2], w22);
        t[2][3] = mul(t[2][3], w23);
        t[3][1] = mul(t[3][1], w13);
        t[3][2] = mul(t[3][2], w23);
        t[3][3] = mul(t[3][3], w33);
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            c32 u[4] = {t[0][k1], t[1][k1], t[2][k1], t[3][k1]};
            Dft<4, S>::run(u);
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = u[k2];
        }
    }
};

template <int S>
struct Dft<32, S> {
    static __device__ __forceinline__ void run(c32 *v)
    {
        // 2 x 16: radix 2 over n1 (n = 16 n1 + n2), twiddle W32^{n2 k1},
        // DFT16 over n2 for each k1; output k = k1 + 2 k2.
        const float c1 = 0.98078528040323044913f;  // cos(pi/16)
        const float s1 = 0.19509032201612826785f;  // sin(pi/16)
        const float c2 = 0.92387953251128675613f;  // cos(pi/8)
        const float s2 = 0.38268343236508977173f;  // sin(pi/8)
        const float c3 = 0.83146961230254523708f;  // cos(3 pi/16)
        const float s3 = 0.55557023301960222474f;  // sin(3 pi/16)
        const float r2 = 0.70710678118654752440f;
        // cos and sin of 2 pi m / 32, m = 0 .. 15
        const float cs[16] = {1.f, c1, c2, c3, r2, s3, s2, s1, 0.f, -s1, -s2, -s3, -r2, -c3, -c2, -c1};
        const float sn[16] = {0.f, s1, s2, s3, r2, c3, c2, c1, 1.f, c1, c2, c3, r2, s3, s2, s1};
        c32 e[16], o[16];
#pragma unroll
        for (int n2 = 0; n2 < 16; ++n2) {
            const c32 a = v[n2], b = v[16 + n2];
            e[n2] = add(a, b);
            const c32 d = sub(a, b);
            if (n2 == 0)
                o[n2] = d;
            else if (n2 == 8)
                o[n2] = muli<S>(d);
            else
                o[n2] = mul(d, c32{cs[n2], S * sn[n2]});
        }
        Dft<16, S>::run(e);
        Dft<16, S>::run(o);
#pragma unroll
        for (int k2 = 0; k2 < 16; ++k2) {
            v[2 * k2] = e[k2];
            v[2 * k2 + 1] = o[k2];
        }
    }
};

// ---------------------------------------------------------------- radix plan
// Factors for a line of length L = 2^a * 3^b * 5^c: the power-of-two part in
// ceil(a/4) factors of 2..16 with the bits spread evenly (512 -> 8,8,8;
// 256 -> 16,16; 128 -> 16,8), then the factors 3 and 5.  A stage takes one
// factor, or, where 3s and 5s are more than one, two adjacent ones
// (r = r1 r2) in the same registers: each stage is an exchange through LDS
// with two barriers, and the pair does what its two stages would, value by
// value, without the exchange between them.  Pairs are joined so that the
// stages are fewest, and of those so that the largest stage is smallest
// (360 -> 8*3,3*5; 900 -> 4*3,3*5,5); line_plan says how large they may be
// (registers).  A single
// 3 or 5 stays a stage of its own: joining it (192 as 8,8*3) made those
// passes 0 to 14 % slower (320^3 forward: 163 -> 179 us), the longer
// butterflies leaving too few per tile for its threads.
constexpr int kMaxFactors = 12;
constexpr int kMaxPair = 25;   // largest pair (points) of a plain pass
constexpr int kEpiPair = 16;   // and of the fused last-axis pass

struct RadixPlan {
    int n;                 // stages
    int r[kMaxFactors];    // radix of each stage
    int r1[kMaxFactors];   // its first factor (r1 = r: a single one)
    int nf;                // factors
    int f[kMaxFactors];
    int nodd;              // factors of 3 and 5
};

// Fewest stages from factor i on with stages of at most m points.
__host__ __device__ constexpr int fewest_stages(const RadixPlan &p, int i, int m)
{
    if (i >= p.nf) return 0;
    if (p.f[i] > m) return 1 << 20;
    int best = 1 + fewest_stages(p, i + 1, m);
    if (i + 1 < p.nf && p.f[i] * p.f[i + 1] <= m) {
        const int two = 1 + fewest_stages(p, i + 2, m);
        if (two < best) best = two;
    }
    return best;
}
__host__ __device__ constexpr RadixPlan radix_plan(int L, int cap = kMaxPair)
{
    RadixPlan p{};
    int a = 0;
    while (L % 2 == 0) {
        L /= 2;
        ++a;
    }
    const int ns2 = (a + 3) / 4;
    for (int st = 0; st < ns2; ++st) p.f[p.nf++] = 1 << (a / ns2 + (st < a % ns2 ? 1 : 0));
    for (; L % 3 == 0; L /= 3) p.f[p.nf++] = 3;
    for (; L % 5 == 0; L /= 5) p.f[p.nf++] = 5;
    p.nodd = p.nf - ns2;
    if (p.nodd <= 1) {
        for (; p.n < p.nf; ++p.n) p.r[p.n] = p.r1[p.n] = p.f[p.n];
        return p;
    }
    const int ns = fewest_stages(p, 0, cap);
    int m = 2;
    while (m < cap && fewest_stages(p, 0, m) > ns) ++m;
    for (int i = 0; i < p.nf;) {
        const bool pair = i + 1 < p.nf && p.f[i] * p.f[i + 1] <= m &&
                          p.n + 1 + fewest_stages(p, i + 2, m) == ns;
        p.r1[p.n] = p.f[i];
        p.r[p.n++] = pair ? p.f[i] * p.f[i + 1] : p.f[i];
        i += pair ? 2 : 1;
    }
    return p;
}

// Columns of a narrow strided tile: 64 KiB of LDS at most, >= 128-byte row
// segments up to L = 512.
__host__ __device__ constexpr int s_b(int L)
{
    return L <= 128 ? 64 : L <= 256 ? 32 : L <= 512 ? 16 : L <= 1024 ? 8 : 4;
}

constexpr int kSThreads = 512;  // most threads of a narrow strided tile

// Points of work of a strided tile's line over the stages of p with nt
// threads: each thread takes every js-th of the L / R butterflies of a stage,
// js = nt / columns, so a stage costs ceil((L / R) / js) js R points.
// Butterflies of more than 32 values a thread (registers) do not count.
__host__ __device__ constexpr int s_work(int L, const RadixPlan &p, int nt)
{
    const int js = nt / s_b(L);
    int w = 0;
    for (int st = 0; st < p.n; ++st) {
        const int nb = (L / p.r[st] + js - 1) / js;
        if (nb * p.r[st] > 32) return 1 << 30;
        w += nb * js * p.r[st];
    }
    return w;
}
// Threads of a strided tile: of the whole-wave counts up to 512 the one with
// the least work over the stages, the larger one of equals.  Lines with at
// most one factor of 3 or 5 take 512: powers of two divide evenly over them,
// and the others (320, 384, ...) measured no faster with fewer.
__host__ __device__ constexpr int s_threads(int L, const RadixPlan &p)
{
    if (L < 16 || p.nodd <= 1) return kSThreads;
    int best = kSThreads, work = s_work(L, p, best);
    for (int nt = kSThreads - 64; nt >= 128; nt -= 64) {
        const int w = nt % s_b(L) == 0 ? s_work(L, p, nt) : work;
        if (w < work) {
            best = nt;
            work = w;
        }
    }
    return best;
}

// The plan of a line: pairs of at most CAP points, or of at most 16 where two
// stages of larger pairs leave more than a fifth of the lanes idle (300 as
// 12,25: 0.77 busy with its registers spilled, r2c y pass 57 us at 300^3; as
// 12,5,5: 46).  Pairs of 24 and 25 points need 128 to 150 registers in a
// plain pass and over 200 in the fused one, which then keeps two waves per
// SIMD (216 as 24,9: 90 us at 360 x 300 x 216; as 8,9,3: 71): CAP is 16 there.
template <int CAP>
__host__ __device__ constexpr RadixPlan line_plan(int L)
{
    const RadixPlan p = radix_plan(L, CAP);
    if (p.nodd <= 1 || CAP <= 16) return p;
    return 5 * p.n * L < 4 * s_work(L, p, s_threads(L, p)) ? radix_plan(L, 16) : p;
}
// Evaluated once per length and translation unit.
template <int L, int CAP = kMaxPair>
inline constexpr RadixPlan kPlan = line_plan<CAP>(L);
// Threads of the plain strided tile and of the fused last-axis one.
template <int L>
inline constexpr int s_nt = s_threads(L, kPlan<L>);
template <int L>
inline constexpr int e_nt = s_threads(L, kPlan<L, kEpiPair>);

// ------------------------------------------------------------ column engine
// NL interleaved lines (columns of a strided pass), element (line l, point p)
// at buf[l + p * NL].  NT is a multiple of NL, so thread tid always works on
// line tid % NL and on butterflies j = tid / NL + i * (NT / NL).  The first
// stage may take its inputs straight from global memory (rows j + r L/R of
// the thread's column, which for consecutive lanes are adjacent addresses)
// and the last stage may store its outputs straight to global memory (the
// last stage of a Stockham DIT writes point j + r L/R).  Stages that read
// and write LDS wait at a barrier between their reads and their writes.

// Global loads and stores of one complex value; NTM = true marks them
// nontemporal (streamed past the caches' normal allocation), which pays for
// the long-stride passes whose lines are touched once.
typedef float lf2_f2 __attribute__((ext_vector_type(2)));

template <bool NTM>
__device__ __forceinline__ c32 gload(const c32 *p)
{
    if constexpr (NTM) {
        const lf2_f2 t = __builtin_nontemporal_load((const lf2_f2 *)p);
        return c32{t.x, t.y};
    } else {
        return *p;
    }
}

template <bool NTM>
__device__ __forceinline__ void gstore(c32 *p, c32 v)
{
    if constexpr (NTM) {
        lf2_f2 t;
        t.x = v.x;
        t.y = v.y;
        __builtin_nontemporal_store(t, (lf2_f2 *)p);
    } else {
        *p = v;
    }
}

// Twiddle index r k C (C = L / (NS R), r < R, k < NS, all below 2^24) with
// a 24-bit multiply (full rate) rather than a 32-bit one.
template <int C>
__device__ __forceinline__ int tw_index(int r, int k)
{
    return (int)__umul24((unsigned)k, (unsigned)(r * C));
}

// Points p, p + qs, ..., p + (R - 1) qs of a column (zeros when !gv), and
// the stores back: one 64-bit pointer add per access, no multiplies.
template <int R, bool NTM>
__device__ __forceinline__ void gload_pts(c32 (&v)[R], const c32 *p, int64_t qs, bool gv)
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        v[r] = gv ? gload<NTM>(p) : c32{0.f, 0.f};
        p += qs;
    }
}
template <int R, bool NTM>
__device__ __forceinline__ void gstore_pts(const c32 (&v)[R], c32 *p, int64_t qs)
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        gstore<NTM>(p, v[r]);
        p += qs;
    }
}

// A line whose stages may be pairs (kPlan: more than one factor of 3 or 5).
template <int L>
inline constexpr bool kPaired = kPlan<L>.nodd > 1;

// a w.  Which product of a sum the compiler folds into the fused
// multiply-add is left to it in most stages, and is spelled out here and in
// dft_fixed, so that kernels which run a stage of another kernel's line give
// its bits.  XW: im = fma(a.x, w.y, a.y w.x), as in a compiled line's last
// stage where that stores to memory; else fma(a.y, w.x, a.x w.y), as in its
// other stages and in the run-time-schedule stages (lf2_kgen.hip).
template <bool XW = false>
__device__ __forceinline__ c32 twiddle_mul(c32 a, c32 w)
{
    const float re = fmaf(a.x, w.x, -(a.y * w.y));
    return c32{re, XW ? fmaf(a.x, w.y, a.y * w.x) : fmaf(a.y, w.x, a.x * w.y)};
}

// Dft<R, S>, the sums of two products in the 5- and 16-point ones spelled out
// in the same way: as in the run-time-schedule stages, or (T32) as in the
// compiled ones, which differ in one of the 16-point twiddles.
template <int R, int S, bool T32 = false>
__device__ __forceinline__ void dft_fixed(c32 *v)
{
    if constexpr (R == 5) {
        const float c1 = 0.30901699437494742410f;   // cos(2 pi / 5)
        const float c2 = -0.80901699437494742410f;  // cos(4 pi / 5)
        const float s1 = 0.95105651629515357212f;   // sin(2 pi / 5)
        const float s2 = 0.58778525229247312917f;   // sin(4 pi / 5)
        const c32 t1 = add(v[1], v[4]), t2 = add(v[2], v[3]);
        const c32 t3 = sub(v[1], v[4]), t4 = sub(v[2], v[3]);
        const c32 a0 = v[0];
        const c32 m1 = c32{fmaf(c2, t2.x, fmaf(c1, t1.x, a0.x)), fmaf(c2, t2.y, fmaf(c1, t1.y, a0.y))};
        const c32 m2 = c32{fmaf(c1, t2.x, fmaf(c2, t1.x, a0.x)), fmaf(c1, t2.y, fmaf(c2, t1.y, a0.y))};
        const c32 n1 = muli<S>(c32{fmaf(s2, t4.x, s1 * t3.x), fmaf(s2, t4.y, s1 * t3.y)});
        const c32 n2 = muli<S>(c32{fmaf(s2, t3.x, -(s1 * t4.x)), fmaf(s2, t3.y, -(s1 * t4.y))});
        v[0] = add(a0, add(t1, t2));
        v[1] = add(m1, n1);
        v[4] = sub(m1, n1);
        v[2] = add(m2, n2);
        v[3] = sub(m2, n2);
    } else if constexpr (R == 16) {
        const float c1 = 0.92387953251128675613f;  // cos(pi/8)
        const float s1 = 0.38268343236508977173f;  // sin(pi/8)
        const float r2 = 0.70710678118654752440f;
        c32 t[4][4];
#pragma unroll
        for (int n2 = 0; n2 < 4; ++n2) {
#pragma unroll
            for (int n1 = 0; n1 < 4; ++n1) t[n2][n1] = v[4 * n1 + n2];
            Dft<4, S>::run(t[n2]);
        }
        auto m = [](c32 a, c32 w) {
            return c32{fmaf(-a.y, w.y, a.x * w.x), fmaf(a.y, w.x, a.x * w.y)};
        };
        auto my = [](c32 a, c32 w) {
            return c32{fmaf(a.x, w.x, -(a.y * w.y)), fmaf(a.x, w.y, a.y * w.x)};
        };
        const c32 w11 = c32{c1, S * s1}, w12 = c32{r2, S * r2}, w13 = c32{s1, S * c1};
        const c32 w23 = c32{-r2, S * r2}, w33 = c32{-c1, -S * s1};
        t[1][1] = m(t[1][1], w11);
        t[1][2] = m(t[1][2], w12);
        t[1][3] = m(t[1][3], w13);
        t[2][1] = m(t[2][1], w12);
        t[2][2] = muli<S>(t[2][2]);
        t[2][3] = m(t[2][3], w23);
        t[3][1] = m(t[3][1], w13);
        t[3][2] = T32 ? my(t[3][2], w23) : m(t[3][2], w23);
        const c32 a = t[3][3];
        t[3][3] = c32{fmaf(a.x, w33.x, -(a.y * w33.y)), fmaf(a.x, w33.y, a.y * w33.x)};
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            c32 u[4] = {t[0][k1], t[1][k1], t[2][k1], t[3][k1]};
            Dft<4, S>::run(u);
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = u[k2];
        }
    } else {
        Dft<R, S>::run(v);
    }
}

// The stage twiddles and the radix-R butterfly of the thread's values v
// (points j + r L/R, k = j mod NS) of a kPaired line.  R = R1 R2: the R2
// butterflies of radix R1 over the points r2 + R2 r1 (twiddles
// W_{NS R1}^{r1 k}), then, where R2 > 1, the R1 butterflies of radix R2 that
// the next stage would do on their outputs (k + r1 NS there: twiddles
// W_{NS R}^{r2 (k + r1 NS)}); output r1 + R1 r2 of the pair is output r of a
// radix-R stage.
template <int L, int R, int R1, int NS, int S>
__device__ __forceinline__ void butterfly(c32 (&v)[R], int k, const c32 *tw)
{
    constexpr int R2 = R / R1;
    static_assert(R1 * R2 == R, "two factors at most");
    c32 t[R2][R1];
#pragma unroll
    for (int r2 = 0; r2 < R2; ++r2) {
#pragma unroll
        for (int r1 = 0; r1 < R1; ++r1) {
            t[r2][r1] = v[r2 + R2 * r1];
            if (NS > 1 && r1 > 0) {
                c32 w = tw[tw_index<L / (NS * R1)>(r1, k)];
                if (S > 0) w = conjg(w);
                t[r2][r1] = twiddle_mul(t[r2][r1], w);
            }
        }
        dft_fixed<R1, S>(t[r2]);
    }
#pragma unroll
    for (int r1 = 0; r1 < R1; ++r1) {
        c32 u[R2];
#pragma unroll
        for (int r2 = 0; r2 < R2; ++r2) {
            u[r2] = t[r2][r1];
            if (r2 > 0 && (NS > 1 || r1 > 0)) {
                c32 w = tw[tw_index<L / (NS * R)>(r2, k + r1 * NS)];
                if (S > 0) w = conjg(w);
                u[r2] = twiddle_mul(u[r2], w);
            }
        }
        if constexpr (R2 > 1) dft_fixed<R2, S>(u);
#pragma unroll
        for (int r2 = 0; r2 < R2; ++r2) v[r1 + R1 * r2] = u[r2];
    }
}

// The butterfly of a first stage (no twiddles before it).
template <int L, int R, int R1, int S>
__device__ __forceinline__ void dft_first(c32 (&v)[R], const c32 *tw)
{
    if constexpr (kPaired<L>)
        butterfly<L, R, R1, 1, S>(v, 0, tw);
    else
        Dft<R, S>::run(v);
}

// A first stage's hooks: on the values of a butterfly it loads from memory
// (row engine), and between its loads and its butterflies.
struct NoHook {
    template <int R>
    __device__ __forceinline__ void values(const c32 (&)[R]) const {}
    __device__ __forceinline__ void loaded() const {}
};

template <int L, int R, int R1, int NS, int S, int NL, int NT, bool SRC_G, bool DST_G, bool NTM = false,
          class Hook = NoHook>
__device__ __forceinline__ void col_stage(c32 *buf, const c32 *gin, c32 *gout, int64_t gs,
                                          bool gv, const c32 *tw, int tid, Hook hook = {})
{
    constexpr int Q = L / R;
    constexpr int JS = NT / NL;
    constexpr int NB = (Q + JS - 1) / JS;
    static_assert(NT % NL == 0, "threads must tile the lines");
    static_assert(!DST_G || NS * R == L, "only the last stage stores to global memory");
    const int l = tid % NL;
    const int j0 = tid / NL;
    c32 v[NB][R];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int j = j0 + i * JS;
        if (Q % JS == 0 || j < Q) {
            if (SRC_G) {
                // (a column past the end is column 0; its loads at 1024 points and
                // more are not conditional, since the compiler waited for the first
                // of them: 80 x 192 x 1024 z back 48.0 us, 45.8 without.  Forward they
                // are, where P(k) rests on the bits)
                gload_pts<R, NTM>(v[i], gin + (int64_t)j * gs, (int64_t)Q * gs,
                                  gv || (L >= 1024 && S > 0));
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) v[i][r] = buf[l + (j + r * Q) * NL];
            }
        }
    }
    hook.loaded();
    if (!SRC_G && !DST_G) __syncthreads();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int j = j0 + i * JS;
        if (Q % JS == 0 || j < Q) {
            const int k = j % NS;
            if constexpr (kPaired<L>) {
                butterfly<L, R, R1, NS, S>(v[i], k, tw);
            } else {
                if (NS > 1) {
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        c32 w = tw[tw_index<L / (NS * R)>(r, k)];
                        if (S > 0) w = conjg(w);
                        v[i][r] = mul(v[i][r], w);
                    }
                }
                Dft<R, S>::run(v[i]);
            }
            if (DST_G) {
                if (gv) gstore_pts<R, NTM>(v[i], gout + (int64_t)j * gs, (int64_t)Q * gs);
            } else {
                c32 *dst = buf + l + ((j / NS) * NS * R + k) * NL;
#pragma unroll
                for (int r = 0; r < R; ++r) dst[r * NS * NL] = v[i][r];
            }
        }
    }
    if (!DST_G) __syncthreads();
}

// ------------------------------------------------------------ row engine
// RB rows of NC interleaved components (the x pass): component c of point p
// of row q sits at global offset at(q) + p * NC + c (RowAt) and at
// buf[(q * NC + c) * LP + lpad(p)] in LDS (one LDS line per row and
// component).  lpad inserts one empty slot after every 16 points, so the
// stride-R writes of the early Stockham stages (points j R + r over
// consecutive j) fall in different banks; LP must be at least
// lpad(points per line - 1) + 1 (row_pitch).
// Butterfly b = tid + i NT of a stage maps to component b % NC, then
// j = (b / NC) % Q, then row b / (NC Q): consecutive lanes walk consecutive
// memory, so the first stage's global loads (point j + r Q) and the last
// stage's global stores are contiguous across a wave.  Only rows < nvalid
// exist in memory.
// PACK (real rows of the r2c / c2r x pass): the global side is a float
// array with row offsets in floats, and point p of component c is the pair
// (f[2p][c], f[2p + 1][c]) = floats (2p) NC + c and (2p + 1) NC + c, loaded
// (first stage) or stored (last stage) as two floats.

// Element offset of row q of a tile: rows y0 + q of plane z0 on, n1 rows a
// plane.  Where planes follow each other like rows (flat), a multiply;
// computed where it is used, since a table of them in LDS had to be filled
// and waited for before a tile's first load.
struct RowAt {
    int64_t base, row, plane;
    uint32_t y0, n1;
    bool flat;
    __device__ __forceinline__ int64_t operator()(int q) const
    {
        if (flat) return base + (int64_t)q * row;
        uint32_t y = y0 + (uint32_t)q, dz = 0;
        if (y >= n1) {  // past the tile's first plane; past its second, divide
            y -= n1;
            dz = 1;
            if (y >= n1) {
                const uint32_t d = y / n1;
                dz += d;
                y -= d * n1;
            }
        }
        return base + (int64_t)dz * plane + (int64_t)y * row;
    }
};
// The same from a table in LDS.
struct RowTable {
    const int64_t *at;
    __device__ __forceinline__ int64_t operator()(int q) const { return at[q]; }
};
__device__ __forceinline__ RowAt row_at(int64_t off, int64_t row, int64_t plane, int n1, int64_t r0)
{
    RowAt a;
    const uint32_t z0 = (uint32_t)r0 / (uint32_t)n1;  // fewer than 2^31 rows
    a.row = row;
    a.plane = plane;
    a.n1 = (uint32_t)n1;
    a.y0 = (uint32_t)r0 - z0 * a.n1;
    a.flat = plane == row * n1;
    a.base = off + (int64_t)z0 * plane + (a.flat ? (int64_t)a.y0 * row : 0);
    return a;
}

__host__ __device__ constexpr int lpad(int p) { return p + (p >> 4); }
__host__ __device__ constexpr int row_pitch(int npoints) { return lpad(npoints - 1) + 1; }

template <bool NTM>
__device__ __forceinline__ float gloadf(const float *p)
{
    if constexpr (NTM)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

template <bool NTM>
__device__ __forceinline__ void gstoref(float *p, float v)
{
    if constexpr (NTM)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

template <int L, int R, int R1, int NS, int S, int RB, int NC, int LP, int NT, bool SRC_G, bool DST_G,
          bool NTM = false, bool PACK = false, class AtI, class AtO, class Hook = NoHook>
__device__ __forceinline__ void row_stage(c32 *buf, const c32 *gin, c32 *gout, const AtI &in_at,
                                          const AtO &out_at, int nvalid, const c32 *tw, int tid,
                                          Hook hook = {})
{
    constexpr int Q = L / R;
    constexpr int NBF = RB * NC * Q;
    constexpr int NB = (NBF + NT - 1) / NT;
    static_assert(!DST_G || NS * R == L, "only the last stage stores to global memory");
    c32 v[NB][R];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int b = tid + i * NT;
        if (NBF % NT == 0 || b < NBF) {
            const int c = b % NC, t = b / NC;
            const int j = t % Q, q = t / Q;
            const int l = q * NC + c;
            // a row past the last one loads the last, and is neither summed nor
            // stored: loads under a condition were joined by register copies,
            // each of which waited for its load (complex x passes, us: 16 x 192 x
            // 1024 back 42.6 and 28.5, 16 x 192 x 768 with six components 68.8 and
            // 61.5, 512 x 96 x 6 with three forward 11.6 and 10.6).  Not the forward
            // pass over one complex component, which has no such copies and
            // whose bits P(k) of a field rests on.
            constexpr bool kClamp = PACK || NC > 1 || S > 0;
            const int64_t at = SRC_G ? in_at(!kClamp || q < nvalid ? q : nvalid - 1) : 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (SRC_G && PACK) {
                    const float *fp = (const float *)gin + at + 2 * (j + r * Q) * NC + c;
                    v[i][r] = c32{gloadf<NTM>(fp), gloadf<NTM>(fp + NC)};
                } else if (SRC_G) {
                    const c32 *p = gin + at + (j + r * Q) * NC + c;
                    v[i][r] = kClamp || q < nvalid ? gload<NTM>(p) : c32{0.f, 0.f};
                } else {
                    v[i][r] = buf[l * LP + lpad(j + r * Q)];
                }
            }
            if (SRC_G && q < nvalid) hook.values(v[i]);
        }
    }
    hook.loaded();
    if (!SRC_G && !DST_G) __syncthreads();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int b = tid + i * NT;
        if (NBF % NT == 0 || b < NBF) {
            const int c = b % NC, t = b / NC;
            const int j = t % Q, q = t / Q;
            const int l = q * NC + c;
            const int k = j % NS;
            const int64_t at = DST_G ? out_at(q) : 0;
            if constexpr (kPaired<L>) {
                butterfly<L, R, R1, NS, S>(v[i], k, tw);
            } else {
                if (NS > 1) {
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        c32 w = tw[tw_index<L / (NS * R)>(r, k)];
                        if (S > 0) w = conjg(w);
                        v[i][r] = mul(v[i][r], w);
                    }
                }
                Dft<R, S>::run(v[i]);
            }
            if (DST_G && PACK) {
                if (q < nvalid) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        float *fp = (float *)gout + at + 2 * (j + r * Q) * NC + c;
                        gstoref<NTM>(fp, v[i][r].x);
                        gstoref<NTM>(fp + NC, v[i][r].y);
                    }
                }
            } else if (DST_G) {
                if (q < nvalid) {
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        gstore<NTM>(gout + at + (j + r * Q) * NC + c, v[i][r]);
                }
            } else {
                c32 *dst = buf + l * LP;
                const int p0 = (j / NS) * NS * R + k;
#pragma unroll
                for (int r = 0; r < R; ++r) dst[lpad(p0 + r * NS)] = v[i][r];
            }
        }
    }
    if (!DST_G) __syncthreads();
}

template <int L, int S, int RB, int NC, int LP, int NT, bool SRC_G, bool DST_G, int ST = 0,
          int NS = 1, bool NTM = false, bool PACK = false, class AtI, class AtO, class Hook = NoHook>
__device__ __forceinline__ void row_fft(c32 *buf, const c32 *gin, c32 *gout, const AtI &in_at,
                                        const AtO &out_at, int nvalid, const c32 *tw, int tid,
                                        Hook hook = {})
{
    if constexpr (L == 1) {
        hook.loaded();
        for (int b = tid; b < RB * NC; b += NT) {
            const int c = b % NC, q = b / NC;
            c32 v = buf[b * LP];
            if (SRC_G && PACK) {
                const float *fp = (const float *)gin + in_at(q) + c;
                v = q < nvalid ? c32{fp[0], fp[NC]} : c32{0.f, 0.f};
            } else if (SRC_G) {
                v = q < nvalid ? gin[in_at(q) + c] : c32{0.f, 0.f};
            }
            if (SRC_G) {
                const c32 u[1] = {v};
                hook.values(u);
            }
            if (DST_G && PACK) {
                if (q < nvalid) {
                    float *fp = (float *)gout + out_at(q) + c;
                    fp[0] = v.x;
                    fp[NC] = v.y;
                }
            } else if (DST_G) {
                if (q < nvalid) gout[out_at(q) + c] = v;
            } else {
                buf[b * LP] = v;
            }
        }
        __syncthreads();
    } else if constexpr (NS < L) {
        constexpr int R = kPlan<L>.r[ST], R1 = kPlan<L>.r1[ST];
        constexpr bool first = ST == 0, last = NS * R == L;
        row_stage<L, R, R1, NS, S, RB, NC, LP, NT, first && SRC_G, last && DST_G, NTM, PACK>(
            buf, gin, gout, in_at, out_at, nvalid, tw, tid, hook);
        row_fft<L, S, RB, NC, LP, NT, SRC_G, DST_G, ST + 1, NS * R, NTM, PACK>(
            buf, gin, gout, in_at, out_at, nvalid, tw, tid);
    }
}

// Radix of stage st, in the plan's order or (REV) in reverse order.  Any
// order of the factors gives the same DFT; the reverse order lets a
// transform start with the radix another one ended with (register hand-off
// in the fused Poisson pass).
template <int L, int CAP>
__host__ __device__ constexpr int radix_sel(int st, bool rev)
{
    return kPlan<L, CAP>.r[rev ? kPlan<L, CAP>.n - 1 - st : st];
}
template <int L, int CAP>
__host__ __device__ constexpr int radix1_sel(int st, bool rev)
{
    return kPlan<L, CAP>.r1[rev ? kPlan<L, CAP>.n - 1 - st : st];
}

// Butterflies per thread of a column stage with Q = L / R butterflies per
// line and NT / NL threads per line.
__host__ __device__ constexpr int col_nb(int L, int R, int NL, int NT)
{
    return (L / R + NT / NL - 1) / (NT / NL);
}

// First half of a column stage: load the butterfly inputs (global memory or
// LDS), apply the stage twiddles and the radix-R DFT, and leave the R outputs
// of each butterfly j in v (they belong at points j + r Q when this is the
// last stage).  After LDS reads the block waits at a barrier, so LDS may be
// rewritten afterwards.
template <int L, int R, int R1, int NS, int S, int NL, int NT, bool SRC_G, bool NTM = false>
__device__ __forceinline__ void col_stage_in(const c32 *buf, const c32 *gin, int64_t gs, bool gv,
                                             const c32 *tw, int tid,
                                             c32 (&v)[col_nb(L, R, NL, NT)][R])
{
    constexpr int Q = L / R;
    constexpr int JS = NT / NL;
    constexpr int NB = col_nb(L, R, NL, NT);
    const int l = tid % NL;
    const int j0 = tid / NL;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int j = j0 + i * JS;
        if (Q % JS == 0 || j < Q) {
            if (SRC_G) {
                gload_pts<R, NTM>(v[i], gin + (int64_t)j * gs, (int64_t)Q * gs, gv);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) v[i][r] = buf[l + (j + r * Q) * NL];
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) v[i][r] = c32{0.f, 0.f};
        }
    }
    if (!SRC_G) __syncthreads();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int j = j0 + i * JS;
        const int k = j % NS;
        if constexpr (kPaired<L>) {
            butterfly<L, R, R1, NS, S>(v[i], k, tw);
        } else {
            if (NS > 1) {
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    c32 w = tw[tw_index<L / (NS * R)>(r, k)];
                    if (S > 0) w = conjg(w);
                    v[i][r] = mul(v[i][r], w);
                }
            }
            Dft<R, S>::run(v[i]);
        }
    }
}

// Second half of a column stage: store v (as produced by col_stage_in with
// the same L, R, NS) to global memory (last stage only) or to the LDS slots
// the next stage reads; LDS writes end at a barrier.
template <int L, int R, int NS, int NL, int NT, bool DST_G, bool NTM = false>
__device__ __forceinline__ void col_stage_out(c32 *buf, c32 *gout, int64_t gs, bool gv, int tid,
                                              const c32 (&v)[col_nb(L, R, NL, NT)][R])
{
    constexpr int Q = L / R;
    constexpr int JS = NT / NL;
    constexpr int NB = col_nb(L, R, NL, NT);
    static_assert(!DST_G || NS * R == L, "only the last stage stores to global memory");
    const int l = tid % NL;
    const int j0 = tid / NL;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int j = j0 + i * JS;
        if (Q % JS == 0 || j < Q) {
            const int k = j % NS;
            if (DST_G) {
                if (gv) gstore_pts<R, NTM>(v[i], gout + (int64_t)j * gs, (int64_t)Q * gs);
            } else {
                c32 *dst = buf + l + ((j / NS) * NS * R + k) * NL;
#pragma unroll
                for (int r = 0; r < R; ++r) dst[r * NS * NL] = v[i][r];
            }
        }
    }
    if (!DST_G) __syncthreads();
}

// Whole transform of the NL columns; SRC_G / DST_G select global input for
// the first stage and global output for the last stage.  L = 1 is a copy.
// REV runs the radices in reverse order; SKIP_LAST stops before the last
// stage (whose inputs are then in LDS).
template <int L, int S, int NL, int NT, bool SRC_G, bool DST_G, int ST = 0, int NS = 1,
          bool NTM = false, bool REV = false, bool SKIP_LAST = false, int CAP = kMaxPair,
          class Hook = NoHook>
__device__ __forceinline__ void col_fft(c32 *buf, const c32 *gin, c32 *gout, int64_t gs, bool gv,
                                        const c32 *tw, int tid, Hook hook = {})
{
    if constexpr (L == 1) {
        hook.loaded();
        if (tid < NL) {
            const int l = tid;
            c32 v = SRC_G ? (gv ? gin[0] : c32{0.f, 0.f}) : buf[l];
            if (DST_G) {
                if (gv) gout[0] = v;
            } else {
                buf[l] = v;
            }
        }
        __syncthreads();
    } else if constexpr (NS < L) {
        constexpr int R = radix_sel<L, CAP>(ST, REV), R1 = radix1_sel<L, CAP>(ST, REV);
        constexpr bool first = ST == 0, last = NS * R == L;
        if constexpr (!(last && SKIP_LAST)) {
            col_stage<L, R, R1, NS, S, NL, NT, first && SRC_G, last && DST_G, NTM>(buf, gin, gout, gs,
                                                                               gv, tw, tid, hook);
            col_fft<L, S, NL, NT, SRC_G, DST_G, ST + 1, NS * R, NTM, REV, SKIP_LAST, CAP>(buf, gin, gout,
                                                                                    gs, gv, tw, tid);
        }
    }
}

}  // namespace lf2
