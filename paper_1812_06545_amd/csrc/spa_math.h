// Device arithmetic of the sum-product check rule, shared by every kernel so
// that all decoding paths round identically.
//
// Check rule (arxiv 1812.06545, Section I: belief propagation / sum-product;
// Algorithm 1, Loop 2): r_mn = 2 atanh(prod_{n' != n} tanh(q_mn'/2)).
// Signs and magnitudes separate: sign = prod sign(q_mn'), and the magnitude
// follows from the |q|.  Each kernel evaluates a row as two halves with
// prefix and suffix combinations (never "total minus self" or a division,
// which cancel or fail when one term dominates or is zero), through an
// arithmetic type A that supplies:
//     Term  term(q)        per-edge quantity and q's sign;
//     Acc   identity()     the empty combination;
//     Acc   add(Acc, Term) combination grown by one edge;
//     Acc   merge(Acc, Acc) combination of two disjoint edge sets;
//     Acc   seed(Acc)      a combination in the form message() takes it
//                          (FP32: its product doubled), applied once per
//                          half row to the other half's combination;
//     T     message(Acc)   |r| from the seeded combination of the other
//                          edges, clamped to R_MAX.
//
// FP32 (base-2 LLR units: every LLR is multiplied by log2(e) on entry and by
// ln 2 on exit) uses the product form directly.  An edge carries
//     t = tanh(|q| ln2 / 2) = (1 - e) / (1 + e)   and   u = 1 - t = 2e / (1 + e),
// with e = 2^-|q|, both to relative accuracy (1 - e for small |q| comes from a
// short series instead of the subtraction).  A combination carries the
// product P = prod t and its complement Q = 1 - P, the latter grown by
// a (+) b = a + b - ab = 1 - (1 - a)(1 - b), so that Q stays accurate when P is
// close to 1 (confident rows) just as P does when it is small.  The message
// is 2 atanh(P) = log2((1 + P) / Q) = log2(1 + 2P / Q), with the rounding
// error of w = fl(1 + z) added back (c = (1 - w) + z is exact while w <
// 2^24, and at most 2^-24 for z < 1; it is clamped to that bound, which
// leaves it exact where it matters, weak messages, and harmless elsewhere).
// The factor 2 of 2P rides on the seed of each half's backward pass, so it
// costs one operation per half row, not per edge.  Per edge: exp2 and one
// reciprocal forward, one reciprocal and log2 back.
//
// FP64 uses the same product form in natural LLR units with its own exp and
// log (ArithF64 below), built from the Taylor series: every term and message
// is accurate to a few units in the last place.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ldpc {

// A condition of every lane of the wavefront, as a mask in scalar registers.
// (As a plain condition the compiler recomputes it in vector registers.)
using Lanes = uint64_t;
__device__ __forceinline__ bool lane_of(Lanes m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// The lanes whose value has its sign bit set.
__device__ __forceinline__ Lanes sign_lanes(float v) { return __ballot(__float_as_int(v) < 0); }
__device__ __forceinline__ Lanes sign_lanes(double v) { return __ballot(__double_as_longlong(v) < 0); }

struct ArithF32 {
    using T = float;
    static constexpr float kIn = 1.44269504088896341f;   // natural LLR -> internal (log2 e)
    static constexpr float kOut = 0.693147180559945309f; // internal -> natural LLR (ln 2)
    static constexpr float kRmax = 28.8539008177792681f; // R_MAX = 20 in internal units

    struct Term {
        float t;   // tanh(|q| ln2 / 2)
        float u;   // 1 - t
        Lanes neg;  // q's sign bit, of all lanes
    };
    struct Acc {
        float P;  // product of the t
        float Q;  // 1 - P, formed from the u
    };
    // a (+) b = 1 - (1 - a)(1 - b) for a, b in [0, 1]
    __device__ static __forceinline__ float oplus(float a, float b) { return __builtin_fmaf(-a, b, a + b); }

    __device__ static __forceinline__ Acc identity() { return Acc{1.0f, 0.0f}; }
    __device__ static __forceinline__ Term term(float q)
    {
        const float x = __builtin_fabsf(q);
        const float e = __builtin_amdgcn_exp2f(-x);
        // d = 1 - 2^-x.  For small x the subtraction loses relative accuracy,
        // which t (a small factor of P, the size of a weak message) needs;
        // there d comes from the Taylor series of -expm1(-x ln 2) (5 terms:
        // truncation below 1e-8 relative for x < 1/8).
        // Everything is formed at half scale, d/2 and 2/(1 + e), which
        // scales by powers of two only (the same roundings) and saves the
        // doubling of e in u = 2e/(1 + e).
        float c5 = 0.5f * 1.33335581e-3f;  // ln2^5/120
        // in a register: an instruction that holds the constant itself cannot
        // take |q|, and x would cost an instruction of its own
        asm("" : "+s"(c5));
        float p = __builtin_fmaf(-x, c5, 0.5f * 9.61812911e-3f);  // ln2^4/24
        p = __builtin_fmaf(-x, p, 0.5f * 5.55041087e-2f);            // ln2^3/6
        p = __builtin_fmaf(-x, p, 0.5f * 2.40226507e-1f);                             // ln2^2/2
        p = __builtin_fmaf(-x, p, 0.5f * 6.93147181e-1f);                             // ln2
        float series = x * p;
        // a select, not a branch around one of its values: a row stays one block
        // of code, whose edges' chains overlap
        asm("" : "+v"(series));
        const float dh = x < 0.125f ? series : __builtin_fmaf(e, -0.5f, 0.5f);  // d / 2
        const float ri2 = __builtin_amdgcn_rcpf(__builtin_fmaf(e, 0.5f, 0.5f));     // 2 / (1 + e)
        Term k;
        k.t = dh * ri2;
        k.u = e * ri2;
        k.neg = sign_lanes(q);
        return k;
    }
    __device__ static __forceinline__ Acc add(Acc a, const Term &k)
    {
        return Acc{a.P * k.t, oplus(a.Q, k.u)};
    }
    __device__ static __forceinline__ Acc merge(Acc a, Acc b) { return Acc{a.P * b.P, oplus(a.Q, b.Q)}; }
    __device__ static __forceinline__ Acc seed(Acc a) { return Acc{a.P + a.P, a.Q}; }
    __device__ static __forceinline__ float message(Acc x)
    {
        // x.P is twice the product (seed).  Q = 0 (a degree-1 row, or every
        // other edge certain) gives z = +inf, w = +inf and log2 = +inf; c is
        // then NaN or a clamp bound, and either way r is not below R_MAX, so
        // the final select (false for NaN) returns R_MAX.  P = 0 forces Q = 1,
        // so z is never 0 * inf.
        const float z = x.P * __builtin_amdgcn_rcpf(x.Q);
        const float w = 1.0f + z;
        const float c = __builtin_amdgcn_fmed3f((1.0f - w) + z, -0x1p-24f, 0x1p-24f);
        const float r = __builtin_fmaf(c, 1.44269504088896341f, __builtin_amdgcn_logf(w));
        return r < kRmax ? r : kRmax;
    }
};

// FP64, natural LLR units, the product form of ArithF32: t = (1 - e)/(1 + e),
// u = 2e/(1 + e) with e = exp(-|q|), message log1p(2P/Q).  One range
// reduction |q| = k ln 2 - r and one series of expm1(r) give both e =
// 2^-k (1 + expm1 r) and 1 - e = (1 - 2^-k) - 2^-k expm1 r to relative
// accuracy (k = 0 leaves -expm1 r itself), and one reciprocal serves t and u.
// Bound by FP64 issue (a v_fma_f64 holds its SIMD 4.9 cycles, v_rcp_f64
// 16.2): about 75 such operations per edge and iteration.  The phi form it
// replaced, r = phi(sum phi(|q|)) with phi(x) = log1p(2 e^-x / -expm1(-x)),
// took six library calls and two divisions per edge.  Fused decodes in FP64,
// phi form and this one: 1000 (3,6)-regular frames of n = 504 397 and 172 us,
// 500 qc frames of n = 1944 over 10 iterations 1944 and 690 us; plain 1000
// frames of n = 504 553 and 302 us.  Worst message error over random rows of
// degree 2 to 21 against 80-bit arithmetic: 5.8e-14 and 2.7e-15 relative.
struct ArithF64 {
    using T = double;
    static constexpr double kIn = 1.0;
    static constexpr double kOut = 1.0;
    static constexpr double kRmax = 20.0;

    struct Term {
        double t;  // tanh(|q| / 2)
        double u;  // 1 - t
        Lanes neg;  // q's sign bit, of all lanes
    };
    struct Acc {
        double P;  // product of the t
        double Q;  // 1 - P, formed from the u
    };
    __device__ static __forceinline__ double oplus(double a, double b) { return __builtin_fma(-a, b, a + b); }
    // 1 / x to about an ulp: the hardware's estimate and two Newton steps
    // (x = 0 and overflowing estimates give NaN, which message() turns into R_MAX).
    __device__ static __forceinline__ double recip(double x)
    {
        double y = __builtin_amdgcn_rcp(x);
        y = __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
        return __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
    }
    // ln 2 in two parts: kLn2Hi has 32 significant bits, so k * kLn2Hi is exact for k < 2^21.
    static constexpr double kLn2Hi = 0x1.62e42feep-1, kLn2Lo = 0x1.a39ef35793c76p-33;

    // log1p(z) for z >= 0 (any value once the result exceeds kRmax; NaN for NaN).
    // w = fl(1 + z), c its rounding error, w = 2^k (1 + f) with 1 + f in
    // [sqrt(1/2), sqrt(2)), log(1 + f) = 2 atanh(s) with s = f / (2 + f),
    // |s| < 0.1716: ten terms of the series leave a truncation below 1e-17.
    __device__ static __forceinline__ double log1p_pos(double z)
    {
        const double w = 1.0 + z;
        const double c = (1.0 - w) + z;
        double f = __builtin_amdgcn_frexp_mant(w);  // [1/2, 1)
        int k = __builtin_amdgcn_frexp_exp(w);
        const bool low = f < 0.70710678118654752;
        f = low ? f + f : f;
        k = low ? k - 1 : k;
        f -= 1.0;
        const double s = f * recip(2.0 + f);
        const double v = s * s;
        double p = 2.0 / 21.0;
        p = __builtin_fma(v, p, 2.0 / 19.0);
        p = __builtin_fma(v, p, 2.0 / 17.0);
        p = __builtin_fma(v, p, 2.0 / 15.0);
        p = __builtin_fma(v, p, 2.0 / 13.0);
        p = __builtin_fma(v, p, 2.0 / 11.0);
        p = __builtin_fma(v, p, 2.0 / 9.0);
        p = __builtin_fma(v, p, 2.0 / 7.0);
        p = __builtin_fma(v, p, 2.0 / 5.0);
        p = __builtin_fma(v, p, 2.0 / 3.0);
        const double kd = static_cast<double>(k);
        // 2 s + s v p = f - s (f - v p): f is exact, so the sum's error is that of a small correction
        double wi = __builtin_amdgcn_rcp(w);
        wi = __builtin_fma(wi, __builtin_fma(-w, wi, 1.0), wi);
        double lo = __builtin_fma(kd, kLn2Lo, c * wi);
        lo = lo - s * (f - v * p);
        return __builtin_fma(kd, kLn2Hi, f + lo);
    }

    __device__ static __forceinline__ Acc identity() { return Acc{1.0, 0.0}; }
    __device__ static __forceinline__ Term term(double q)
    {
        // past 800 (and for a dummy edge's +inf) e is 0: t = 1 and u = 0 exactly
        const double x = __builtin_fmin(__builtin_fabs(q), 800.0);
        const double kd = __builtin_rint(x * 1.4426950408889634);
        const int k = static_cast<int>(kd);
        const double r = __builtin_fma(kd, kLn2Lo, __builtin_fma(kd, kLn2Hi, -x));  // -x = r - k ln 2, |r| < 0.347
        double p = 1.0 / 6227020800.0;  // 1/13!
        p = __builtin_fma(r, p, 1.0 / 479001600.0);
        p = __builtin_fma(r, p, 1.0 / 39916800.0);
        p = __builtin_fma(r, p, 1.0 / 3628800.0);
        p = __builtin_fma(r, p, 1.0 / 362880.0);
        p = __builtin_fma(r, p, 1.0 / 40320.0);
        p = __builtin_fma(r, p, 1.0 / 5040.0);
        p = __builtin_fma(r, p, 1.0 / 720.0);
        p = __builtin_fma(r, p, 1.0 / 120.0);
        p = __builtin_fma(r, p, 1.0 / 24.0);
        p = __builtin_fma(r, p, 1.0 / 6.0);
        p = __builtin_fma(r, p, 0.5);
        const double m = __builtin_fma(r * r, p, r);        // expm1(r)
        const double two = __builtin_amdgcn_ldexp(1.0, -k);  // 2^-k, 0 past the range
        const double e = __builtin_fma(two, m, two);
        const double d = __builtin_fma(-two, m, 1.0 - two);
        const double ri = recip(1.0 + e);
        Term out;
        out.t = d * ri;
        out.u = (e + e) * ri;
        out.neg = sign_lanes(q);
        return out;
    }
    __device__ static __forceinline__ Acc add(Acc a, const Term &k)
    {
        return Acc{a.P * k.t, oplus(a.Q, k.u)};
    }
    __device__ static __forceinline__ Acc merge(Acc a, Acc b) { return Acc{a.P * b.P, oplus(a.Q, b.Q)}; }
    __device__ static __forceinline__ Acc seed(Acc a) { return Acc{a.P + a.P, a.Q}; }
    __device__ static __forceinline__ double message(Acc x)
    {
        // Q = 0 gives NaN, which the select turns into R_MAX.
        const double r = log1p_pos(x.P * recip(x.Q));
        return r < kRmax ? r : kRmax;
    }
};

// Exclusive combinations of one check row.  The row's d edges are split at
// h = ceil(d/2) into halves H0 = [0, h) and H1 = [h, d); for edge k in half
// H, with p_k the combination of the earlier edges of H (left to right),
// C_other the combination of the other half (left to right) and s_k the
// combination seed(C_other) grown by the later edges of H (right to left),
//     excl_k = merge(p_k, s_k).
// Fixing the order lets the fused kernel spread a row over two lanes (one
// half each, exchanging C and the sign) while the streaming kernels evaluate
// the same expression in one lane, bit for bit.

// Layered rows (Section II, Algorithm 2; both layered paths) split each half
// once more, into quarters Q0 = [0, q1), Q1 = [q1, h), Q2 = [h, q3) and
// Q3 = [q3, d), with h = ceil(d/2), q1 = ceil(h/2), q3 = h + ceil((d - h)/2).
// For edge k in Qi, excl_k = merge(p_k, s_k) as above, with p_k the
// combination of the earlier edges of Qi and s_k = seed(O_i) grown by its
// later edges, where O_i combines the other three quarters (C_j, each left
// to right) in this fixed association:
//     O_0 = merge(C_1, merge(C_2, C_3))    O_1 = merge(C_0, merge(C_2, C_3))
//     O_2 = merge(C_3, merge(C_0, C_1))    O_3 = merge(C_2, merge(C_0, C_1))
// merge is commutative bit for bit (a product, and a (+) b, whose fused
// multiply-add forms the exact product either way) but not associative.  The
// fused kernel spreads a layered row over four lanes, one quarter each, which
// halves the serial length of a layer step; the streaming layer kernel
// evaluates the same expressions in one lane.
struct Quarters {
    int q1, h, q3;
};
__host__ __device__ constexpr Quarters quarters(int d)
{
    return Quarters{((d + 1) / 2 + 1) / 2, (d + 1) / 2, (d + 1) / 2 + (d - (d + 1) / 2 + 1) / 2};
}
__host__ __device__ constexpr int quarter_of(const Quarters &q, int k)
{
    return k < q.q1 ? 0 : k < q.h ? 1 : k < q.q3 ? 2 : 3;
}

// seed(O_i) for the four quarters from their combinations C.
template <class A>
__device__ __forceinline__ void quarter_seeds(const typename A::Acc C[4], typename A::Acc S[4])
{
    const typename A::Acc c01 = A::merge(C[0], C[1]), c23 = A::merge(C[2], C[3]);
    S[0] = A::seed(A::merge(C[1], c23));
    S[1] = A::seed(A::merge(C[0], c23));
    S[2] = A::seed(A::merge(C[3], c01));
    S[3] = A::seed(A::merge(C[2], c01));
}

// Forward step for an edge with incoming message q: its term a_k, p_k = the
// half's running combination, which then grows by a_k.
template <class A>
__device__ __forceinline__ void check_forward(typename A::T q, typename A::Term &a_k, typename A::Acc &p_k,
                                              typename A::Acc &acc, Lanes &sign)
{
    a_k = A::term(q);
    p_k = acc;
    acc = A::add(acc, a_k);
    sign ^= a_k.neg;
}

// Backward step: outgoing message of an edge from its term, p_k, the half's
// running suffix s (started at seed(C_other); it then grows by this edge) and
// the row's total sign.  Signs are lane masks: a comparison forward and a
// select backward per edge, where a sign carried in t's sign bit cost four
// vector instructions.
// (Leaving out the merges with the identity at a part's first edge saves
// four instructions per half row, but the rows then take 115 registers instead
// of 90 and ran 2-6% slower.)
template <class A>
__device__ __forceinline__ typename A::T check_backward(const typename A::Term &a_k, const typename A::Acc &p_k,
                                                        typename A::Acc &s, Lanes sign_total)
{
    const typename A::Acc ex = A::merge(p_k, s);
    s = A::add(s, a_k);
    const typename A::T mag = A::message(ex);
    return lane_of(sign_total ^ a_k.neg) ? -mag : mag;
}

}  // namespace ldpc
