// The full-window step at N = 4 (M = 2) on entries held in registers, shared by
// the tile kernel (quapi_tile.hip) and the persistent kernel (quapi_small.hip):
// the influence rows and their coefficients, one step on the 16 values of a
// lane, the LDS slots of an exchange and the reduction of rho terms by MFMA.
#pragma once

#include "quapi_device.h"

namespace quapi {
namespace {

// The influence rows of the two off-diagonal points.  For M = 2 and the pair
// o = 1 (s_0, s_1), D = s_0 - s_1 and a lag of coefficient eta,
//   F(1, p) = e^{-i phi} { e^{-i theta}, e^{-g}, e^{g}, e^{i theta} },   p = 0 .. 3,
// phi = D Im(eta) (s_0 + s_1), theta = D^2 Im(eta), g = D^2 Re(eta), and
// F(2, p) the conjugate with p = 1, 2 swapped.  With the phase e^{-i phi} moved
// into the factor tables a row takes four real coefficients:
//   sum_p = cos(theta) (x0 + x3) -+ i sin(theta) (x0 - x3) + e^{-+g} x1 + e^{+-g} x2,
// 8 real multiply-adds instead of 16, and x0 + x3 serves the diagonal rows too.
//
// Coefficients, read by scalar loads, 8 bytes of room each: cos, sin, e^{-g},
// e^{g} of the oldest point (lag L; interior, final class) in the compute
// precision, packed from the start; then in FP64 in every tier, at their index:
// the same of the group digit at lag L-1 (stages 0 and 2, "pair 0"); for the
// group digit e at lag 1, with K (stages 1 and 3, "pair 1"), per stage and e the
// complex factors of o = 1, 2 (interior), then the final class; then per stage
// and e K[0][e], K[3][e].  The stages differ in K for a driven system only.
//
// With FP32 arithmetic an entry's whole factor (outer digits, thread digits,
// group digit) is formed in FP64 and rounded once, and a lane's rho terms are
// FP64 products and sums of FP32 values: every rounding of a factor acts again
// at each step.  rms of rho against complex128 over 120 steps, factors and terms
// in FP32 -> this: L = 8 .. 11 9.9e-8 -> 7.6e-8 (the two-step kernel 8.8e-8),
// L = 5 .. 7 7.8e-8 -> 5.4e-8; it takes 6% of a step at L = 15.
constexpr int kTcOld = 0, kTcOldf = 4, kTcE = 8, kTcEf = 12, kTcLag1 = 16;
__device__ __forceinline__ constexpr int tc_lag1(int stage) { return kTcLag1 + 32 * (stage >> 1); }
__device__ __forceinline__ constexpr int tc_k(int stage) { return kTileCoefK + 16 * stage; }

__device__ __forceinline__ constexpr int mirror_d(int d) { return d == 1 ? 2 : d == 2 ? 1 : d; }

__device__ __forceinline__ int tile_tab(const BankLayout &B, int lag, int cls) {
    if (lag == 1) return cls ? B.k_fin1() : B.k_lag1();
    return cls ? B.fin(lag) : B.lag(lag);
}
// F(mirror(o), mirror(p)) = conj(F(o, p)) bit for bit (the bank's K has it to
// rounding), so that an entry and its mirror come out exactly conjugate.
// entry(t, o, p): the bank's table t.
template <typename Entry>
__device__ __forceinline__ double2 tab4_of(Entry entry, int t, int row, int col) {
    const int k = row * 4 + col, km = mirror_d(row) * 4 + mirror_d(col), kk = km < k ? km : k;
    double2 v = entry(t, kk / 4, kk % 4);
    if (km < k) v.y = -v.y;
    if (km == k) v.y = 0.0;
    return v;
}
__device__ __forceinline__ double2 tab4(const double2 *bank, int t, int row, int col) {
    return tab4_of([&](int tb, int o, int p) { return bank[(size_t)tb * 16 + o * 4 + p]; }, t, row, col);
}
// Coefficient k (see above) into coef; fp32: the compute precision.
template <typename Entry>
__device__ __forceinline__ void put_coef(void *coef, int k, int L, const double2 *eta, const double *s, Entry entry,
                                         bool fp32) {
    const BankLayout B{L};
    double v;
    if (k < kTcLag1) {
        const double2 et = eta[1 + (k / 4 % 2 ? 2 * L : 0) + (k < kTcE ? L : L - 1)];
        const double D = s[0] - s[1], th = D * D * et.y, g = D * D * et.x;
        v = k % 4 == 0 ? cos(th) : k % 4 == 1 ? sin(th) : exp(k % 4 == 2 ? -g : g);
    } else {
        const bool infl = k < kTileCoefK;               // lag 1, or the diagonal rows of K
        const double2 f = tab4_of(entry, infl ? tile_tab(B, 1, k / 4 % 2) : B.k_lag1(),
                                  infl ? 1 + k / 2 % 2 : k / 2 % 2 * 3,
                                  infl ? (k - kTcLag1) / 8 % 4 : (k - kTileCoefK) / 4 % 4);
        v = k % 2 ? f.y : f.x;
        if (!infl && fp32) v = (float)v;                // exact: the diagonal rows of K are FP32 values
    }
    if (k < kTcE && fp32) ((float *)coef)[k] = (float)v;
    else ((double *)coef)[k] = v;
}
// What the thread's factor of point o carries besides its digits' tables: the
// self factor and the phases e^{-+i phi} of the oldest point and (pair 0) of the
// group digit.
__device__ __forceinline__ double2 prefix4(const double2 *bank, const double2 *eta, const double *s, int L, int o,
                                           int cls, int pair) {
    const BankLayout B{L};
    const double ph = (s[0] - s[1]) * (s[0] + s[1]);
    const double2 *e = eta + 1 + (cls ? 2 * L : 0);
    double sn, cs;
    sincos(ph * (e[L].y + (pair == 0 ? e[L - 1].y : 0.0)), &sn, &cs);
    return cmul(tab4(bank, cls ? B.self_end() : B.self_int(), o, 0), make_double2(cs, o == 1 ? -sn : sn));
}

// 8 bytes per slot: a complex64 value, or one component of a complex128 value
// at a time (a whole one would take twice the LDS, half the waves).
template <typename C> struct XSlot;
template <> struct XSlot<float2> {
    static constexpr int kParts = 1;
    using type = float2;
    static __device__ __forceinline__ float2 get(float2 v, int) { return v; }
    static __device__ __forceinline__ void set(float2 &v, float2 s, int) { v = s; }
};
template <> struct XSlot<double2> {
    static constexpr int kParts = 2;
    using type = double;
    static __device__ __forceinline__ double get(double2 v, int part) { return part ? v.y : v.x; }
    static __device__ __forceinline__ void set(double2 &v, double s, int part) { (part ? v.y : v.x) = s; }
};
// D += E_q B over the wave, E_q the 4x4 matrix with ones in row q (4x4x4
// FP64 MFMA, four blocks): adds the wave's values v, reduced 4 : 1, to the 16
// lanes 16 q .. 16 q + 15 of acc.  Four such calls keep four running sums in
// one register pair, where per-lane sums would take four pairs for every
// stage (and shuffles of each at the end of every tile).
__device__ __forceinline__ double row_add(double acc, double v, int q, int lane) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64((lane & 3) == q ? 1.0 : 0.0, v, acc, 0, 0, 0);
}

// The coefficient pointer through an opaque move: loads through it stay at
// their use instead of being kept live in scalar registers.
template <typename T>
__device__ __forceinline__ const T *fresh_t(const T *p) {
    asm volatile("" : "+s"(p));
    return p;
}

// Wave-uniform read of one coefficient (see coef_ld).
template <typename T>
__device__ __forceinline__ T coef_s(const T *p, int k) {
    return ((const __attribute__((address_space(4))) T *)p)[k];
}
__device__ __forceinline__ double fma_t(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }

// The contraction of the oldest point for o = 1 (SIGN +) or o = 2 (SIGN -):
// p = x0 + x3, q = x0 - x3, coefficients at k.  The terms of x1 and x2 are
// taken in mirrored orders for the two points, so that the mirrored group
// gives the exact conjugate.
template <int SIGN, typename T, typename C>
__device__ __forceinline__ C row12(const T *co, int k, C p, C q, C x1, C x2) {
    const T c = coef_s(co, k), sn = SIGN > 0 ? coef_s(co, k + 1) : -coef_s(co, k + 1);
    const T g1 = coef_s(co, k + 2), g2 = coef_s(co, k + 3);
    const C a = SIGN > 0 ? x1 : x2, b = SIGN > 0 ? x2 : x1;
    C r;
    r.x = fma_t(g2, b.x, fma_t(g1, a.x, fma_t(sn, q.y, c * p.x)));
    r.y = fma_t(g2, b.y, fma_t(g1, a.y, fma_t(-sn, q.x, c * p.y)));
    return r;
}

// K[0][prev] and K[3][prev] of a stage, prev wave-uniform (scalar loads).
template <typename T>
__device__ __forceinline__ void coef_k(const T *coef, int stage, int prev, double2 &k0, double2 &k3) {
    const double *kd = (const double *)fresh_t(coef) + tc_k(stage) + 4 * prev;
    k0 = coef_ld(kd, 0);
    k3 = coef_ld(kd, 1);
}

// One step (stage) on the 16 values of a lane: digit PAIR of the register index
// (stride 4^PAIR) is contracted, the groups are the other digit e.  c1, c2: the
// thread's factors of the new points 1 and 2 (interior); kp0, kp3: K[0][prev] and
// K[3][prev] where the previous point is not e (PAIR 0; see coef_k).  With RHO: tf1, tf2 the
// final-point sums of the lane without the thread's factor, rd0 and rd3 the
// terms of the diagonal points (REAL: their real parts only).
template <typename T, bool RHO, bool REAL, int STAGE, typename CI>
__device__ __forceinline__ void tile_stage(const CI (&in)[16], typename Cx<T>::type (&w)[16],
                                           const T *coef, double2 c1, double2 c2, double2 kp0, double2 kp3,
                                           double2 &tf1, double2 &tf2, double2 &rd0, double2 &rd3) {
    using C = typename Cx<T>::type;
    constexpr int PAIR = STAGE % 2;
    constexpr int SI = PAIR == 0 ? 1 : 4, SE = PAIR == 0 ? 4 : 1;
    const T *co = fresh_t(coef);
    double2 all = make_double2(0.0, 0.0);
    if (RHO) tf1 = tf2 = rd0 = rd3 = make_double2(0.0, 0.0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        __builtin_amdgcn_sched_barrier(0);      // a group at a time: fewer live registers
        const T *ce = PAIR == 0 ? co : fresh_t(coef);
        const C x0 = conv<C>(in[SE * e]), x1 = conv<C>(in[SE * e + SI]);
        const C x2 = conv<C>(in[SE * e + 2 * SI]), x3 = conv<C>(in[SE * e + 3 * SI]);
        const C p = cadd(x0, x3);
        C q;
        q.x = x0.x - x3.x;
        q.y = x0.y - x3.y;
        // the diagonal points 0 and 3 carry no influence: K times the plain sum
        // (K[0][e], K[3][e] are real for e = 0, 3)
        TraceSum<C> sd;
        if constexpr (sizeof(T) == 4) {
            TraceSum<C> s2;
            sd.init(x0);
            sd.add(x3);
            s2.init(x1);
            s2.add(x2);
            sd.s = cadd(sd.s, s2.s);
        } else {
            sd.init(cadd(p, cadd(x1, x2)));
        }
        const double *kd = (const double *)ce + tc_k(STAGE) + 4 * e;
        const double2 d0 = PAIR == 0 ? kp0 : coef_ld(kd, 0), d3 = PAIR == 0 ? kp3 : coef_ld(kd, 1), ds = sd.s;
        if (PAIR == 1 && (e == 0 || e == 3)) {
            w[SE * e] = from_d2<C>(make_double2(d0.x * ds.x, d0.x * ds.y));
            w[SE * e + 3 * SI] = from_d2<C>(make_double2(d3.x * ds.x, d3.x * ds.y));
        } else {
            w[SE * e] = from_d2<C>(cmul(d0, ds));
            w[SE * e + 3 * SI] = from_d2<C>(cmul(d3, ds));
        }
        if (RHO) {
            if (PAIR == 0) {
                all = cadd(all, ds);
            } else if (REAL) {
                rd0.x = fma(d0.x, ds.x, rd0.x);
                rd3.x = fma(d3.x, ds.x, rd3.x);
                if (e == 1 || e == 2) {
                    rd0.x = fma(-d0.y, ds.y, rd0.x);
                    rd3.x = fma(-d3.y, ds.y, rd3.x);
                }
            } else {
                cmac(rd0, d0, ds);
                cmac(rd3, d3, ds);
            }
        }
        // e's own factor: for pair 0 the four-coefficient form of the row
        auto factor_e = [&](int o, bool fin) {
            const double *cd = (const double *)ce;
            double2 f;
            if (PAIR == 0) {
                const int k = fin ? kTcEf : kTcE;
                f.x = coef_s(cd, e == 1 || e == 2 ? k + ((e == 1) == (o == 1) ? 2 : 3) : k);
                f.y = (e == 0) == (o == 1) ? -coef_s(cd, k + 1) : coef_s(cd, k + 1);
            } else {
                const int k = tc_lag1(STAGE) + 8 * e + 2 * (o - 1) + (fin ? 4 : 0);
                f.x = coef_s(cd, k);
                f.y = coef_s(cd, k + 1);
            }
            return f;
        };
        constexpr bool kRealE = PAIR == 0;            // factors of e = 1, 2 are real
        auto with_e = [&](double2 c, int o) {
            const double2 f = factor_e(o, false);
            if (!(kRealE && (e == 1 || e == 2))) return from_d2<C>(cmul(c, f));
            return from_d2<C>(make_double2(c.x * f.x, c.y * f.x));
        };
        auto add_e = [&](double2 &sum, C s, int o) {  // sum += factor * s (final class)
            const double2 f = factor_e(o, true), v = to_d2(s);
            if (kRealE && (e == 1 || e == 2)) {
                sum.x = fma(v.x, f.x, sum.x);
                sum.y = fma(v.y, f.x, sum.y);
            } else {
                cmac(sum, v, f);
            }
        };
        const C s1 = row12<1>(co, kTcOld, p, q, x1, x2), s2 = row12<-1>(co, kTcOld, p, q, x1, x2);
        w[SE * e + SI] = cmul(with_e(c1, 1), s1);
        w[SE * e + 2 * SI] = cmul(with_e(c2, 2), s2);
        if (RHO) {
            add_e(tf1, row12<1>(co, kTcOldf, p, q, x1, x2), 1);
            add_e(tf2, row12<-1>(co, kTcOldf, p, q, x1, x2), 2);
        }
    }
    if (RHO && PAIR == 0) {
        rd0 = cmul(kp0, all);
        rd3 = cmul(kp3, all);
    }
}

}  // namespace
}  // namespace quapi
