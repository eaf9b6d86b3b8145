// The pair term of the sweep: exact cutoff predicate, cubic B-spline kernel
// and its gradient, and the three accumulation precisions.
#pragma once

#include "pi_internal.h"

// Constants of one sweep, derived on the host from rc (= h, the support).
struct KernelConst {
    float lo, hi;       // filter on fl(r^2): < lo surely inside, >= hi surely outside
    float reach2;       // rc^2 and a margin for roundings, rounded up: a cell whose nearest
                        // face is at fl(distance^2) >= reach2 surely holds no pair inside
                        // the cutoff
    double hh64;        // h*h, exact in double
    float hh, eh;       // h*h rounded to float, and its residual: h^2 = hh + eh exactly
    float hh_quarter;   // hh / 4 (exact): r^2 <= hh/4  <=>  q <= 1/2
    float h, inv_h;
    float sigma;        // 8 / (pi h^3)
    float two_sigma;    // 2 sigma
    float sig_h2;       // sigma / h^2        (W'(r)/r = sig_h2 (18 q - 12) for q <= 1/2)
    float six_sig_h;    // 6 sigma / h        (W'(r)   = -six_sig_h (1-q)^2 for q > 1/2)
    float w;            // cell width
    float inv_w;        // 1 / w
    float rc2_cells;    // (rc / w)^2
};

// The arithmetic of a time step with PI_PREC_COMPENSATED: h^2 - r^2 by FP32
// error-free transforms and Kahan-compensated FP32 sums; with PI_PREC_FP64ACC the same
// h^2 - r^2 and FP64 sums of FP32 terms; both as the first time steps of this
// library had them.  A last bit of G that differs moves some
// particles to the next point of the position lattice, and the trajectory leaves
// its earlier course from there (with the FP64 forms below, G differed by up to
// 1.5e-3 of its mean size after eight steps of 2^24 particles): the time steps
// keep their arithmetic, so that a simulation can be taken up and checked against
// earlier runs bit for bit.  In the sub-box tiles at 1 per cell it costs little: 0.79 ms
// of a step of 2^24 particles, 0.78 with the FP64 forms.
constexpr int kPrecStep = 3, kPrecStep64 = 4;
constexpr bool step_precision(int prec) { return prec >= kPrecStep; }

// h^2 - (dx^2 + dy^2 + dz^2) in FP64, which the vector units issue at the rate
// of (non-packed) FP32: the square of a float is exact in double (48
// significant bits), and so is h^2, so the only roundings are the three of
// the FMA chain, each at most 2^-53 h^2 (the partial results are no larger
// than h^2 for every pair inside the cutoff).  The sign is exact whenever
// |h^2 - r^2| exceeds 2^-51 h^2, which holds for every pair of points on a
// power-of-two lattice of spacing >= 2^-22 h; it is tested in double, so a
// tiny difference cannot underflow to zero.  The evaluation of a pair is
// bound by VALU issue, and this takes 7 instructions (three conversions,
// three FMAs, one conversion back) where the same difference by FP32
// error-free transforms took 25.  Sweep kernel times with the transforms and
// with this: 2^24 particles at 1 per cell 1.21 and 1.18 ms, at 8 per cell
// 5.42 and 4.86 ms, 2^23 clustered 5.4 and 4.9 ms; the largest error of an
// output against 64 bits (2-norm) 1.1e-7 and 1.0e-7.
__device__ __forceinline__ double h2_minus_d2(float dx, float dy, float dz, const KernelConst &k)
{
    const double x = (double)dx, y = (double)dy, z = (double)dz;
    return __builtin_fma(-z, z, __builtin_fma(-y, y, __builtin_fma(-x, x, k.hh64)));
}

// Error of a + b = s (Knuth's TwoSum, branch-free): a + b == s + err exactly.
__device__ __forceinline__ float two_sum_err(float a, float b, float s)
{
    const float bb = s - a;
    return (a - (s - bb)) + (b - bb);
}

// The same by error-free transforms in FP32: the squares are split into float +
// exact FMA residual, their sum into float + TwoSum errors, and the large part
// is subtracted from hh exactly (Sterbenz, since the sum is within a factor of
// two of hh wherever this matters).  The sign is exact whenever
// |h^2 - r^2| exceeds about 6 * 2^-48 h^2.
__device__ __forceinline__ float h2_minus_d2_fp32(float dx, float dy, float dz, const KernelConst &k)
{
    const float p1 = dx * dx, e1 = __builtin_fmaf(dx, dx, -p1);
    const float p2 = dy * dy, e2 = __builtin_fmaf(dy, dy, -p2);
    const float p3 = dz * dz, e3 = __builtin_fmaf(dz, dz, -p3);
    const float a = p1 + p2;
    const float t1 = two_sum_err(p1, p2, a);
    const float s = a + p3;
    const float t2 = two_sum_err(a, p3, s);
    const float tail = ((t1 + t2) + (e1 + e2)) + e3; // r^2 = s + tail
    const float head = k.hh - s;
    return head + (k.eh - tail);
}

// Whether h^2 - r^2 > 0, and its value as a term uses it.
template <int PREC>
__device__ __forceinline__ bool h2_above_d2(float dx, float dy, float dz, const KernelConst &k)
{
    if (step_precision(PREC)) return h2_minus_d2_fp32(dx, dy, dz, k) > 0.0f;
    return h2_minus_d2(dx, dy, dz, k) > 0.0;
}

template <int PREC>
__device__ __forceinline__ float h2_minus_d2_term(float dx, float dy, float dz, const KernelConst &k)
{
    if (step_precision(PREC)) return h2_minus_d2_fp32(dx, dy, dz, k);
    return (float)h2_minus_d2(dx, dy, dz, k);
}

// The exact predicate in the band [lo, hi), which almost no candidate falls
// into: the empty asm keeps the compiler from evaluating it for every
// candidate ahead of the branch (cheap enough, in FP64, to be speculated).
template <int PREC>
__device__ __forceinline__ bool in_band_inside(float dx, float dy, float dz, const KernelConst &k)
{
    asm volatile("");
    return h2_above_d2<PREC>(dx, dy, dz, k);
}

// Filtered exact predicate r < rc from the FP32 value t = fl(r^2) computed as
// fma(dz, dz, fma(dy, dy, dx * dx)) (relative error below 3.0001 * 2^-24).
template <int PREC>
__device__ __forceinline__ bool inside_cutoff(float dx, float dy, float dz, float t, const KernelConst &k)
{
    if (t < k.lo) return true;
    if (t >= k.hi) return false;
    return in_band_inside<PREC>(dx, dy, dz, k);
}

__device__ __forceinline__ float sq_dist(float dx, float dy, float dz)
{
    return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

// Kernel value W(r) and W'(r)/r of an accepted pair.  With SELECT both
// pieces of the spline are evaluated and one is chosen, with the same
// values as the branch: where a wavefront evaluates queued pairs together it
// almost always holds pairs on both sides of q = 1/2, so the branch would
// run both anyway (and the merge after it costs register copies).  The
// unchosen piece may be infinite (the outer one at r = 0); it is not used.
template <int PREC, bool SELECT = false>
__device__ __forceinline__ void bspline_terms(float dx, float dy, float dz, float t, const KernelConst &k,
                                              float &W, float &Fr)
{
    const float r = __builtin_amdgcn_sqrtf(t);
    if (SELECT) {
        const float q = r * k.inv_h;
        const float w_in = k.sigma * __builtin_fmaf(q * q, __builtin_fmaf(6.0f, q, -6.0f), 1.0f);
        const float f_in = k.sig_h2 * __builtin_fmaf(18.0f, q, -12.0f);
        float omq;
        if (PREC == PI_PREC_PLAIN) {
            omq = fmaxf(1.0f - r * k.inv_h, 0.0f);
        } else {
            const float D = h2_minus_d2_term<PREC>(dx, dy, dz, k);
            omq = D * __builtin_amdgcn_rcpf(k.h * (k.h + r));
        }
        const float omq2 = omq * omq;
        const float w_out = k.two_sigma * omq2 * omq;
        const float f_out = -k.six_sig_h * omq2 * __builtin_amdgcn_rsqf(t);
        const bool inner = t <= k.hh_quarter;
        W = inner ? w_in : w_out;
        Fr = inner ? f_in : f_out;
        return;
    }
    if (t <= k.hh_quarter) {
        const float q = r * k.inv_h;
        W = k.sigma * __builtin_fmaf(q * q, __builtin_fmaf(6.0f, q, -6.0f), 1.0f);
        Fr = k.sig_h2 * __builtin_fmaf(18.0f, q, -12.0f);
    } else {
        float omq;
        if (PREC == PI_PREC_PLAIN) {
            omq = fmaxf(1.0f - r * k.inv_h, 0.0f);
        } else {
            // 1 - q = (h^2 - r^2) / (h (h + r)), with h^2 - r^2 free of cancellation
            const float D = h2_minus_d2_term<PREC>(dx, dy, dz, k);
            omq = D * __builtin_amdgcn_rcpf(k.h * (k.h + r));
        }
        const float omq2 = omq * omq;
        W = k.two_sigma * omq2 * omq;
        Fr = -k.six_sig_h * omq2 * __builtin_amdgcn_rsqf(t);
    }
}

// Per-target accumulators for rho and G.  An accepted pair adds w_j W to rho
// and f (dx, dy, dz) with f = w_j W'(r) / r to G.
template <int PREC>
struct Acc;

template <>
struct Acc<PI_PREC_PLAIN> {
    float rho = 0.f, gx = 0.f, gy = 0.f, gz = 0.f;
    __device__ __forceinline__ void add(float a, float f, float dx, float dy, float dz)
    {
        rho += a;
        gx += f * dx;
        gy += f * dy;
        gz += f * dz;
    }
    __device__ __forceinline__ float r_rho() const { return rho; }
    __device__ __forceinline__ float r_gx() const { return gx; }
    __device__ __forceinline__ float r_gy() const { return gy; }
    __device__ __forceinline__ float r_gz() const { return gz; }
};

// FP64 sums, with the products f dx not rounded on their own: the error of a
// sum is that of its FP32 terms.  A lane's sums take eight registers, as
// FP32 sums with a compensation term each would, and one pair two
// conversions, an addition and three FMAs in FP64 (the differences are
// already there in FP64, from h^2 - r^2): about 30 cycles, against about 50
// for three products and four Kahan additions in FP32.  Sweep kernel times
// with Kahan sums and with these, 2^24 particles: 8 per cell 4.86 and 4.35 ms,
// 1 per cell 1.18 and 1.16 ms; the largest error of an output against 64 bits
// (2-norm) 1.0e-7 and 9.7e-8.
template <>
struct Acc<PI_PREC_FP64ACC> {
    double rho = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    __device__ __forceinline__ void add(float a, float f, float dx, float dy, float dz)
    {
        const double fd = (double)f;
        rho += (double)a;
        gx = __builtin_fma(fd, (double)dx, gx);
        gy = __builtin_fma(fd, (double)dy, gy);
        gz = __builtin_fma(fd, (double)dz, gz);
    }
    __device__ __forceinline__ float r_rho() const { return (float)rho; }
    __device__ __forceinline__ float r_gx() const { return (float)gx; }
    __device__ __forceinline__ float r_gy() const { return (float)gy; }
    __device__ __forceinline__ float r_gz() const { return (float)gz; }
};

// FP64 sums hold at least what compensated FP32 sums do, and cost less here.
template <>
struct Acc<PI_PREC_COMPENSATED> : Acc<PI_PREC_FP64ACC> {};

// Kahan's compensated summation: c is the rounding excess of the running sum
// so far (what was added minus what was meant), taken off the next term.
template <>
struct Acc<kPrecStep> {
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    float c0 = 0.f, c1 = 0.f, c2 = 0.f, c3 = 0.f;
    __device__ __forceinline__ static void ks(float &s, float &c, float v)
    {
        const float y = v - c;
        const float n = s + y;
        c = (n - s) - y;
        s = n;
    }
    __device__ __forceinline__ void add(float a, float f, float dx, float dy, float dz)
    {
        ks(s0, c0, a);
        ks(s1, c1, f * dx);
        ks(s2, c2, f * dy);
        ks(s3, c3, f * dz);
    }
    __device__ __forceinline__ float r_rho() const { return s0 - c0; }
    __device__ __forceinline__ float r_gx() const { return s1 - c1; }
    __device__ __forceinline__ float r_gy() const { return s2 - c2; }
    __device__ __forceinline__ float r_gz() const { return s3 - c3; }
};

template <>
struct Acc<kPrecStep64> {
    double rho = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    __device__ __forceinline__ void add(float a, float f, float dx, float dy, float dz)
    {
        rho += (double)a;
        gx += (double)(f * dx);
        gy += (double)(f * dy);
        gz += (double)(f * dz);
    }
    __device__ __forceinline__ float r_rho() const { return (float)rho; }
    __device__ __forceinline__ float r_gx() const { return (float)gx; }
    __device__ __forceinline__ float r_gy() const { return (float)gy; }
    __device__ __forceinline__ float r_gz() const { return (float)gz; }
};

// Everything a target keeps while it walks its 27 cells.
template <int PREC, bool INV>
struct Target {
    Acc<PREC> acc;
    int32_t count = 0;
    float ascale = 0.f; // sum w_j |W'(r)| (only with INV)

    // One candidate source at offset (dx, dy, dz) = x_i - x_j, weight wj.
    __device__ __forceinline__ void candidate(float dx, float dy, float dz, float wj, const KernelConst &k)
    {
        const float t = sq_dist(dx, dy, dz);
        if (t < k.hi && inside_cutoff<PREC>(dx, dy, dz, t, k)) accept(dx, dy, dz, t, wj, k);
    }

    // The same for a wavefront that evaluates queued pairs together: every lane
    // runs, and a lane whose `ok` is false adds zeros, which change no sum (its
    // differences must be finite).  One straight piece of code: accumulators
    // that a branch carries cost a register copy each per round.  The selects are
    // the compiler's: it keeps two wait states between the compare that writes a
    // lane mask and the select that reads it, which it would not around one
    // written in inline assembly.  Sweep kernels with these, and with assembly
    // that held the waits itself: 2^24 particles at 1 per cell (7x7x5) 0.80 and
    // 0.80 ms, at 8 per cell 2.41 and 2.48, 2^21 at 64 per cell 1.97 and 2.03.
    __device__ __forceinline__ void pair_if(bool ok, float dx, float dy, float dz, float t, float wj,
                                            const KernelConst &k)
    {
        float W, Fr;
        bspline_terms<PREC, true>(dx, dy, dz, t, k, W, Fr);
        // (the products, not a factor: either may be infinite; and chosen as
        // floats, not after the conversion, which the empty asm is for)
        float a = ok ? wj * W : 0.0f, f = ok ? wj * Fr : 0.0f;
        asm("" : "+v"(a), "+v"(f));
        // (adding zero would move a Kahan sum's excess into the sum)
        if (PREC != kPrecStep || ok) acc.add(a, f, dx, dy, dz);
        count += ok ? 1 : 0;
        if (INV) ascale += -f * __builtin_amdgcn_sqrtf(t); // (Fr <= 0)
    }

    template <bool SELECT = false>
    __device__ __forceinline__ void accept(float dx, float dy, float dz, float t, float wj, const KernelConst &k)
    {
        float W, Fr;
        bspline_terms<PREC, SELECT>(dx, dy, dz, t, k, W, Fr);
        const float f = wj * Fr;
        acc.add(wj * W, f, dx, dy, dz);
        count += 1;
        if (INV) ascale += -f * __builtin_amdgcn_sqrtf(t); // w_j |W'|: Fr <= 0
    }
};
