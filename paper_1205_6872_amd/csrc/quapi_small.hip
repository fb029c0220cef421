// Persistent propagation of small tensors: one workgroup per context runs
// every step of a call in one launch, and one launch serves a batch of
// contexts (same N and precision; each block its own context, memory length
// and step range).
//
// Method: Dattani 2012, Sec. II (exact path-sum equation, discretized
// influence functional); the tensor-propagator recursion of the Introduction,
// with rho(t_n) from the final-point classes (Sec. IV 'allPoints' /
// 'justFinalPoint').  The same steps as the multi-block kernels -- growth
// while the window fills, then multiply by K and the new point's factors and
// sum out the oldest point -- but the whole step sequence stays inside one
// workgroup, so a step costs a barrier rather than three kernel launches.
// Two kernels: small_reg_kernel keeps the tensor of M = 2, L = 5..7 in the
// block's registers (full-window steps; in a mixed batch it also takes shorter
// memory lengths); small_kernel runs everything else (growth, other N and L),
// its tensor ping-ponging between two LDS buffers when
// both fit (N^L up to 4096 at complex128), else between the context's two
// global buffers, which stay in the L2 cache at these sizes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "quapi_internal.h"
#include "quapi_step4.h"

namespace quapi {
namespace {

// threads per block: 16 waves where the registers allow (N <= 9), else 4
template <int N> struct SmallBlock {
    static constexpr int threads = N <= 9 ? 1024 : 256;
    static constexpr int waves = threads / 64;
};

__host__ __device__ inline long long ipow_s(int b, int e) {
    long long r = 1;
    for (int i = 0; i < e; ++i) r *= b;
    return r;
}

// LDS layout of one block: the two tensor buffers (in-LDS mode), the
// full-window factor products over the low and high digits of m, interior
// and final ([N][RL], [N][RH] each, compute precision), the oldest-point
// tables (first / main full-window step, interior / final: 4 x [N][N],
// compute precision), and the per-wave rho sums (two parities).
struct SmallLds {
    unsigned buf0, buf1, plo, phi, pflo, pfhi, old, red, total;
    int dlo, dhi, RL, RH;
};
__host__ __device__ inline SmallLds small_lds_layout(int N, int csize_store, int csize_comp, int L, bool in_lds) {
    const int waves = N <= 9 ? SmallBlock<4>::waves : SmallBlock<16>::waves;
    SmallLds l;
    const int nd = L - 1;
    l.dlo = nd / 2;
    l.dhi = nd - l.dlo;
    l.RL = (int)ipow_s(N, l.dlo);
    l.RH = (int)ipow_s(N, l.dhi);
    const unsigned E = (unsigned)ipow_s(N, L);
    unsigned off = 0;
    l.buf0 = lds_take(off, in_lds ? E * csize_store : 0);
    l.buf1 = lds_take(off, in_lds ? E * csize_store : 0);
    l.plo = lds_take(off, N * l.RL * csize_comp);
    l.phi = lds_take(off, N * l.RH * csize_comp);
    l.pflo = lds_take(off, N * l.RL * csize_comp);
    l.pfhi = lds_take(off, N * l.RH * csize_comp);
    l.old = lds_take(off, 4 * N * N * csize_comp);
    l.red = lds_take(off, 2 * waves * N * 16);
    l.total = off;
    return l;
}

// Sum over the 64 lanes of a wave of P values per lane (P a power of two <= 64),
// leaving lane l with the total of value o = l >> (6 - log2 P): a butterfly
// that halves the values each lane carries per round (the half it does not
// keep goes to its partner), then sums the one value left over the lanes that
// share it -- P - 1 + 6 - log2 P exchanges instead of 6 P.
template <int P, int HALF>
__device__ __forceinline__ void scatter_round(double2 (&v)[P], int lane, int d) {
    if constexpr (HALF >= 1) {
        const bool up = (lane & d) != 0;
#pragma unroll
        for (int j = 0; j < HALF; ++j) {
            const double2 send = up ? v[j] : v[j + HALF];
            const double2 keep = up ? v[j + HALF] : v[j];
            v[j].x = keep.x + __shfl_xor(send.x, d, 64);
            v[j].y = keep.y + __shfl_xor(send.y, d, 64);
        }
        scatter_round<P, HALF / 2>(v, lane, d / 2);
    }
}
template <int P>
__device__ __forceinline__ double2 wave_sum_scatter(double2 (&v)[P], int lane) {
    scatter_round<P, P / 2>(v, lane, 32);
    double2 r = v[0];
    for (int d = 32 / P; d >= 1; d /= 2) {
        r.x += __shfl_xor(r.x, d, 64);
        r.y += __shfl_xor(r.y, d, 64);
    }
    return r;
}

// Product over the digits j0 .. j0+nd-1 of v (base N, least significant
// first, digit j of v is table tab(j0 + k)) of the bank tables, row o (FP64).
template <int N, typename TabOf>
__device__ double2 small_digit_product(const double2 *__restrict__ bank, TabOf tab, int j0, int nd, long long v,
                                       int o) {
    double2 p = make_double2(1.0, 0.0);
    for (int k = 0; k < nd; ++k) {
        const int dg = (int)(v % N);
        v /= N;
        p = cmul(p, bank[(size_t)tab(j0 + k) * (N * N) + o * N + dg]);
    }
    return p;
}

// One context's steps by a block of kSB threads.
template <int N, typename S, typename T, bool IN_LDS, int kSB>
__device__ __forceinline__ void small_body(const SmallCtxArgs &a, unsigned char *smem) {
    constexpr int kSW = kSB / 64;
    using C = typename Cx<T>::type;
    using CS = typename Cx<S>::type;
    constexpr int M = N == 1 ? 1 : N == 4 ? 2 : N == 9 ? 3 : 4;
    const int L = a.L;
    const BankLayout B{L};
    const SmallLds lay = small_lds_layout(N, (int)sizeof(CS), (int)sizeof(C), L, IN_LDS);
    C *s_plo = (C *)(smem + lay.plo);
    C *s_phi = (C *)(smem + lay.phi);
    C *s_pflo = (C *)(smem + lay.pflo);
    C *s_pfhi = (C *)(smem + lay.pfhi);
    C *s_old = (C *)(smem + lay.old);          // [4][N][N]: old_first, old_main, oldf_first, oldf_main
    double2 *s_red = (double2 *)(smem + lay.red);
    const double2 *__restrict__ bank = a.bank;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const long long NM = ipow_s(N, L - 1);      // items of a full-window step

    CS *buf[2];
    if (IN_LDS) {
        buf[0] = (CS *)(smem + lay.buf0);
        buf[1] = (CS *)(smem + lay.buf1);
        const long long E0 = ipow_s(N, min(a.step0 + 1, L));
        const CS *src = (const CS *)a.a0;
        for (long long x = t; x < E0; x += kSB) buf[0][x] = src[x];
    } else {
        buf[0] = (CS *)a.a0;
        buf[1] = (CS *)a.a1;
    }
    // the oldest-point tables of every full-window step, and the factor
    // products over the digits of m (formed in FP64, rounded once)
    const int otab[4] = {B.old_first(), B.old_main(), B.oldf_first(), B.oldf_main()};
    for (int idx = t; idx < 4 * N * N; idx += kSB)
        s_old[idx] = from_d2<C>(bank[(size_t)otab[idx / (N * N)] * (N * N) + idx % (N * N)]);
    auto tab_int = [&](int j) { const int lag = L - 1 - j; return lag == 1 ? B.k_lag1() : B.lag(lag); };
    auto tab_fin = [&](int j) { const int lag = L - 1 - j; return lag == 1 ? B.k_fin1() : B.fin(lag); };
    for (int idx = t; idx < N * lay.RL; idx += kSB) {
        const int o = idx / lay.RL, v = idx % lay.RL;
        s_plo[idx] = from_d2<C>(small_digit_product<N>(bank, tab_int, 0, lay.dlo, v, o));
        s_pflo[idx] = from_d2<C>(small_digit_product<N>(bank, tab_fin, 0, lay.dlo, v, o));
    }
    for (int idx = t; idx < N * lay.RH; idx += kSB) {
        const int o = idx / lay.RH, v = idx % lay.RH;
        s_phi[idx] = from_d2<C>(small_digit_product<N>(bank, tab_int, lay.dlo, lay.dhi, v, o));
        s_pfhi[idx] = from_d2<C>(small_digit_product<N>(bank, tab_fin, lay.dlo, lay.dhi, v, o));
    }
    __syncthreads();

    int n_out = 0;
    for (int k = 0; k < a.n_steps; ++k) {
        const int n = a.step0 + 1 + k;
        const bool sel = a.rho_mode == 1 || (a.rho_mode == 2 && k == a.n_steps - 1);
        const CS *__restrict__ in = buf[k & 1];
        CS *__restrict__ out = buf[(k + 1) & 1];
        // waves that own items this step (the others add nothing to rho)
        const long long items = n < L ? ipow_s(N, n) : NM;
        const int nw = (int)min((long long)kSW, (items + 63) / 64);
        double2 acc[N];
#pragma unroll
        for (int o = 0; o < N; ++o) acc[o] = make_double2(0.0, 0.0);
        if (n < L) {
            // growth: points 0 .. n-1 in, n+1 points out; out[x + E_in o] = x F(o, x)
            const long long E_in = ipow_s(N, n);
            auto tab_g = [&](int j) {
                if (j == 0) return n == 1 ? B.k_init1() : B.init(n);
                const int lag = n - j;
                return lag == 1 ? B.k_lag1() : B.lag(lag);
            };
            auto tab_gf = [&](int j) {
                if (j == 0) return n == 1 ? B.k_fin_init1() : B.fin_init(n);
                const int lag = n - j;
                return lag == 1 ? B.k_fin1() : B.fin(lag);
            };
            for (long long x = t; x < E_in; x += kSB) {
                const C xv = conv<C>(in[x]);
                const double2 xd = to_d2(xv);
                // N = 4: the products of every o and both classes run digit by
                // digit together, so that their reads are in flight at once, and
                // the diagonal points take the lag-1 digit's factor only, which
                // carries K (the others are one): a call of the first L steps,
                // M = 2, complex128, L = 7 106 -> 78 us, L = 5 45 -> 41.  (At
                // N = 9, 16 the products held at once spill.)
                double2 p4[N == 4 ? 4 : 1], pf4[N == 4 ? 4 : 1];
                if constexpr (N == 4) {
                    p4[1] = p4[2] = pf4[1] = pf4[2] = make_double2(1.0, 0.0);
                    long long v = x;
                    for (int j = 0; j < n; ++j, v >>= 2) {
                        const double2 *q = bank + tab_g(j) * 16 + (int)(v & 3);
                        const double2 *qf = bank + tab_gf(j) * 16 + (int)(v & 3);
                        const double2 q1 = q[4], q2 = q[8];
                        if (sel) {
                            pf4[1] = cmul(pf4[1], qf[4]);
                            pf4[2] = cmul(pf4[2], qf[8]);
                        }
                        p4[1] = cmul(p4[1], q1);
                        p4[2] = cmul(p4[2], q2);
                        if (j == n - 1) {
                            p4[0] = q[0];
                            p4[3] = q[12];
                            pf4[0] = qf[0];
                            pf4[3] = qf[12];
                        }
                    }
                }
#pragma unroll
                for (int o = 0; o < N; ++o) {
                    double2 f;
                    if constexpr (N == 4) f = p4[o];
                    else f = small_digit_product<N>(bank, tab_g, 0, n, x, o);
                    f = cmul(f, bank[(size_t)B.self_int() * (N * N) + o * N]);
                    out[x + E_in * o] = conv<CS>(cmul(xv, from_d2<C>(f)));
                    if (sel) {
                        double2 ff;
                        if constexpr (N == 4) ff = pf4[o];
                        else ff = small_digit_product<N>(bank, tab_gf, 0, n, x, o);
                        ff = cmul(ff, bank[(size_t)B.self_end() * (N * N) + o * N]);
                        const double2 v = cmul(xd, ff);
                        acc[o].x += v.x;
                        acc[o].y += v.y;
                    }
                }
            }
        } else {
            // full window: out[m + NM o] = P(o, m) sum_i old[o][i] in[i + N m]
            const C *old = s_old + (n == L ? 0 : 1) * N * N;
            const C *oldf = s_old + (n == L ? 2 : 3) * N * N;
            for (long long m = t; m < NM; m += kSB) {
                C x[N];
#pragma unroll
                for (int i = 0; i < N; ++i) x[i] = conv<C>(in[i + N * m]);
                const int ml = (int)(m % lay.RL), mh = (int)(m / lay.RL);
#pragma unroll
                for (int o = 0; o < N; ++o) {
                    const C p = cmul(s_plo[o * lay.RL + ml], s_phi[o * lay.RH + mh]);
                    C v;
                    if (sizeof(T) == 4 && N > 1 && o % (M + 1) == 0 && L >= 2) {
                        // a diagonal point: its oldest-point row is ones and p is
                        // K[o, m_last]; the sum stays unrounded until the product
                        TraceSum<C> ts;
                        ts.init(x[0]);
#pragma unroll
                        for (int i = 1; i < N; ++i) ts.add(x[i]);
                        v = ts.times_right(p);
                    } else {
                        C s = {};
#pragma unroll
                        for (int i = 0; i < N; ++i) cmac(s, old[o * N + i], x[i]);
                        v = cmul(s, p);
                    }
                    out[m + NM * o] = conv<CS>(v);
                    if (sel) {
                        C sf = {};
#pragma unroll
                        for (int i = 0; i < N; ++i) cmac(sf, oldf[o * N + i], x[i]);
                        const C pf = cmul(s_pflo[o * lay.RL + ml], s_pfhi[o * lay.RH + mh]);
                        const double2 w = to_d2(cmul(sf, pf));
                        acc[o].x += w.x;
                        acc[o].y += w.y;
                    }
                }
            }
        }
        if (sel && wave < nw) {
            constexpr int P = N == 1 ? 1 : N <= 4 ? 4 : 16;      // N rounded up to a power of two
            constexpr int lg = P == 1 ? 0 : P == 4 ? 2 : 4;
            double2 v[P];
#pragma unroll
            for (int o = 0; o < P; ++o) v[o] = o < N ? acc[o] : make_double2(0.0, 0.0);
            const double2 r = wave_sum_scatter<P>(v, lane);
            const int o = lane >> (6 - lg);
            double2 *red = s_red + (k & 1) * kSW * N;
            if ((lane & ((64 >> lg) - 1)) == 0 && o < N) red[wave * N + o] = r;
        }
        __syncthreads();          // the new tensor and the wave sums are complete
        if (sel) {
            const double2 *red = s_red + (k & 1) * kSW * N;
            if (t < N) {
                double2 s = make_double2(0.0, 0.0);
                for (int w = 0; w < nw; ++w) {
                    s.x += red[w * N + t].x;
                    s.y += red[w * N + t].y;
                }
                a.rho_out[(size_t)n_out * N + t] = s;
            }
            ++n_out;
        }
    }
    if (IN_LDS) {
        // the last tensor goes to the buffer a step-by-step run would have
        // left it in: a0 after an even number of steps, a1 after an odd one
        const int last = a.step0 + a.n_steps;
        const long long E = ipow_s(N, min(last + 1, L));
        CS *dst = (CS *)((a.n_steps & 1) ? a.a1 : a.a0);
        const CS *src = buf[a.n_steps & 1];
        for (long long x = t; x < E; x += kSB) dst[x] = src[x];
    }
}

template <int N, typename S, typename T, bool IN_LDS>
__global__ void __launch_bounds__(SmallBlock<N>::threads) small_kernel(const SmallBatchArgs args) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SmallCtxArgs a = args.c[blockIdx.x];
    small_body<N, S, T, IN_LDS, SmallBlock<N>::threads>(a, smem);
}

// ------------------------------------------------ the window in registers
// Full-window steps n > L of an M = 2 context with L = 5, 6 or 7, all steps of a
// call in one launch: the tensor stays in the registers of one block, 16 entries
// per thread (4^(L-2) threads), the two oldest points in a thread's registers.
// Two steps contract those; one exchange through LDS then moves the next two
// oldest points into the registers.  A thread's digits stand for the same ages
// at every pair of steps, so its factors never change.  Pairs are fixed by the
// global step number, (L+1, L+2), (L+3, L+4), ...: a call may begin or end inside
// one, and every entry and every rho is formed by the same operations.
//
// Bound by the instructions of one compute unit, about 320 per stage and wave, and
// the exchange.  Before, the tensor went through LDS, or at L = 7 through HBM
// buffers (512 KB a step through one compute unit's L2 port), one item at a time.
// One context, rho at every step / at the last, us per step, before -> now:
//   L = 7  complex128 10.7 / 6.4 -> 4.3 / 2.9   complex64 7.8 / 4.3 -> 4.1 / 2.7
//   L = 6              4.0 / 2.1 -> 1.5 / 1.0              3.0 / 1.4 -> 1.5 / 0.9
//   L = 5              2.0 / 1.0 -> 1.3 / 0.8              1.9 / 0.9 -> 1.4 / 0.8
// At L = 4 (16 columns, a quarter of a wave) a step would gain nothing.
constexpr int kRegSets = 8;              // (stage, class, o in {1, 2})
// A thread stands for U of the 4^(L-2) columns of 16 entries.  U = 2 at L = 7: 1024
// threads leave 128 registers each, of which FP64 values alone take 64 (spilled:
// 17.3 us per step).
template <int L> struct SmallReg {
    static constexpr int cols = 1 << (2 * (L - 2)), U = L == 7 ? 2 : 1;
    static constexpr int threads = cols / U, waves = threads / 64;
    static constexpr int hi = 1 << (2 * (L - 4));            // values of the column's digits above the lowest two
    static constexpr unsigned buf = cols * 16 * 8;           // exchange: 8 bytes per slot
    static constexpr unsigned lds = buf + kRegSets * (16 + hi) * 16 + 2 * 2 * waves * 8 * 8;
};
// The slot of entry y (canonical index) is y ^ reg_bits(y): consecutive lanes'
// 8-byte accesses cover the banks both at y = c + columns r (written) and at
// y = r + 16 c (read).
__device__ __forceinline__ constexpr int reg_bits(int y) { return (y >> 5) & 15; }

template <int L, typename S, typename T>
__device__ __forceinline__ void reg_body(const SmallCtxArgs &a, unsigned char *smem) {
    using C = typename Cx<T>::type;
    using CS = typename Cx<S>::type;
    using X = XSlot<C>;
    using R = SmallReg<L>;
    constexpr int TH = R::threads, U = R::U;
    typename X::type *s_x = (typename X::type *)smem;
    double2 *s_lo = (double2 *)(smem + R::buf);              // [set][16]
    double2 *s_hi = s_lo + kRegSets * 16;                          // [set][hi]
    double *s_red = (double *)(s_hi + kRegSets * R::hi);     // [pair parity][stage][wave][8]
    int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const BankLayout B{L};
    const T *coef = (const T *)a.coef;
    // factors over the thread's digits d2 .. d_(L-1), the lowest two (with the
    // prefix) and the others, in FP64
    for (int idx = t; idx < kRegSets * (16 + R::hi); idx += TH) {
        const bool lo = idx < kRegSets * 16;
        const int k = lo ? idx : idx - kRegSets * 16, q = lo ? k / 16 : k / R::hi;
        const int st = q / 4, cls = q / 2 % 2, o = 1 + q % 2;
        int v = lo ? k % 16 : k % R::hi;
        double2 p = lo ? prefix4(a.bank, a.eta, a.s, L, o, cls, st) : make_double2(1.0, 0.0);
        for (int j = lo ? 0 : 2; j < (lo ? 2 : L - 2); ++j, v >>= 2)
            p = cmul(p, tab4(a.bank, tile_tab(B, L - 2 - j + st, cls), o, v & 3));
        (lo ? s_lo : s_hi)[k] = p;
    }
    // the previous point of a pair's first step is the highest digit of the column
    auto prev_k = [&](int c, double2 &k0, double2 &k3) {
        const int prev = c >> (2 * (L - 3));
        if (L >= 6) {
            coef_k(coef, 0, __builtin_amdgcn_readfirstlane(prev), k0, k3);
        } else {
            const double2 *kd = (const double2 *)((const double *)coef + tc_k(0) + 4 * prev);
            k0 = kd[0];
            k3 = kd[1];
        }
    };
    auto factor = [&](int q, int c) { return cmul(s_lo[q * 16 + (c & 15)], s_hi[q * R::hi + (c >> 4)]); };
    int stage = (a.step0 - L) & 1;                           // of the next step
    // the index of register r's entry: after a pair (or before the first), and
    // after its first step (registers: new point, second oldest)
    auto index = [&](int c, int r) { return stage ? (r >> 2) + 4 * c + (r & 3) * (R::cols * 4) : r + 16 * c; };
    C w[U][16];
    {
        const CS *src = (const CS *)a.a0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) w[u][r] = conv<C>(src[index(t + TH * u, r)]);
    }
    __syncthreads();                                         // every entry is read, the factors are there
    int n_out = 0, par = 0, pend = 0;                        // pend: steps whose wave sums wait in s_red
    double2 *out = a.rho_out;
    auto flush = [&]() {                                     // after a barrier that follows the wave sums
        if (t < 8)
            for (int st = 0; st < 2; ++st)
                if (pend >> st & 1) {
                    const double *p = s_red + (par * 2 + st) * R::waves * 8 + t;
                    double v = 0.0;
                    for (int k = 0; k < R::waves; ++k) v += p[k * 8];
                    ((double *)(out + (size_t)n_out * 4))[t] = v;
                    ++n_out;
                }
        if (t >= 8) n_out += (pend & 1) + (pend >> 1);
        pend = 0;
        par ^= 1;
    };
    // the wave's sums of one step: rows v0.x, v0.y, v1.x, v1.y (s0) and v2, v3 (s1)
    auto add_rho = [&](int st, int c, double2 tf1, double2 tf2, double2 v0, double2 v3, double &s0, double &s1) {
        const double2 v1 = cmul(factor(4 * st + 2, c), tf1), v2 = cmul(factor(4 * st + 3, c), tf2);
        s0 = row_add(s0, v0.x, 0, lane);
        s0 = row_add(s0, v0.y, 1, lane);
        s0 = row_add(s0, v1.x, 2, lane);
        s0 = row_add(s0, v1.y, 3, lane);
        s1 = row_add(s1, v2.x, 0, lane);
        s1 = row_add(s1, v2.y, 1, lane);
        s1 = row_add(s1, v3.x, 2, lane);
        s1 = row_add(s1, v3.y, 3, lane);
    };
    auto put_rho = [&](int st, double s0, double s1) {
        for (int off = 8; off > 0; off >>= 1) {
            s0 += __shfl_xor(s0, off, 64);
            s1 += __shfl_xor(s1, off, 64);
        }
        if ((lane & 15) == 0) {
            double *p = s_red + ((par * 2 + st) * R::waves + wave) * 8;
            p[lane >> 4] = s0;
            p[4 + (lane >> 4)] = s1;
        }
        pend |= 1 << st;
    };
    // one step; STAGE 0 or 1 of the pair
    auto step = [&](auto stage_c, bool sel) {
        constexpr int ST = decltype(stage_c)::value;
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = t + TH * u;
            double2 tf1, tf2, rd0, rd3, k0{}, k3{};
            __builtin_amdgcn_sched_barrier(0);
            if (ST == 0) prev_k(c, k0, k3);
            if (sel) {
                tile_stage<T, true, false, ST>(w[u], w[u], coef, factor(4 * ST, c), factor(4 * ST + 1, c), k0, k3, tf1,
                                               tf2, rd0, rd3);
                add_rho(ST, c, tf1, tf2, rd0, rd3, s0, s1);
            } else {
                tile_stage<T, false, false, ST>(w[u], w[u], coef, factor(4 * ST, c), factor(4 * ST + 1, c), k0, k3,
                                                tf1, tf2, rd0, rd3);
            }
            if (sizeof(S) < sizeof(T)) {                     // a call may end after any step
#pragma unroll
                for (int r = 0; r < 16; ++r) w[u][r] = conv<C>(conv<CS>(w[u][r]));
            }
        }
        if (sel) put_rho(ST, s0, s1);
    };
    auto selected = [&](int k) { return a.rho_mode == 1 || (a.rho_mode == 2 && k == a.n_steps - 1); };
    for (int k = 0; k < a.n_steps; ++k) {                    // a pair, or the part of it in this call
        // opaque per pair: the LDS slots and factors of a thread are formed or read
        // again at each, not kept in registers over the run
        asm volatile("" : "+v"(t));
        if (stage == 0) {
            step(std::integral_constant<int, 0>{}, selected(k));
            stage = 1;
            if (++k >= a.n_steps) break;
        }
        step(std::integral_constant<int, 1>{}, selected(k));
        stage = 0;
        // the next two oldest points into the registers: written at
        // y = column + columns (new points), read at y = r + 16 column
#pragma unroll
        for (int part = 0; part < X::kParts; ++part) {
            __syncthreads();
            if (part == 0) flush();
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    s_x[(t ^ (reg_bits((t & 511) + R::cols * r))) + TH * u + R::cols * r] = X::get(w[u][r], part);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) X::set(w[u][r], s_x[16 * t + 16 * TH * u + (r ^ ((t >> 1) & 15))], part);
        }
    }
    __syncthreads();
    flush();
    CS *dst = (CS *)((a.n_steps & 1) ? a.a1 : a.a0);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[index(t + TH * u, r)] = conv<CS>(w[u][r]);
}

// A block per context, each with the threads of its own memory length (the
// waves beyond them end at once; a barrier waits for those that are left): one
// launch takes as long as its slowest context.  In a batch of other lengths it
// also runs, whole, the contexts of L < kRegMinL, whose full-window steps have
// at most 64 items: one wave.  A call of 150 steps on 24 contexts, complex64, rho
// at every step, a launch per length -> this: L = 5, 6 552 -> 354 us, L = 4, 5
// 584 -> 378, L = 3 .. 6 814 -> 390; one length alone the same (complex128, L = 7
// 766 -> 750).
constexpr int kRegThreads = SmallReg<kRegMaxL>::threads;
constexpr int reg_threads(int L) {
    return L == 7 ? SmallReg<7>::threads : L == 6 ? SmallReg<6>::threads : L == 5 ? SmallReg<5>::threads : 64;
}
template <typename S, typename T>
__global__ void __launch_bounds__(kRegThreads) small_reg_kernel(const SmallBatchArgs args) {
    extern __shared__ __align__(16) unsigned char smem[];
    const SmallCtxArgs &a = args.c[blockIdx.x];
    if ((int)threadIdx.x >= reg_threads(a.L)) return;
    switch (a.L) {
    case 7: reg_body<7, S, T>(a, smem); break;
    case 6: reg_body<6, S, T>(a, smem); break;
    case 5: reg_body<5, S, T>(a, smem); break;
    default: small_body<4, S, T, true, 64>(a, smem); break;
    }
}

template <int N, typename S, typename T>
hipError_t launch_small_t(bool in_lds, const SmallBatchArgs &b, int n_ctx, int L_max, hipStream_t st) {
    const SmallLds lay = small_lds_layout(N, (int)sizeof(typename Cx<S>::type), (int)sizeof(typename Cx<T>::type),
                                          L_max, in_lds);
    if (in_lds)
        hipLaunchKernelGGL((small_kernel<N, S, T, true>), dim3(n_ctx), dim3(SmallBlock<N>::threads), lay.total, st, b);
    else
        hipLaunchKernelGGL((small_kernel<N, S, T, false>), dim3(n_ctx), dim3(SmallBlock<N>::threads), lay.total, st,
                           b);
    return hipGetLastError();
}

template <int N>
hipError_t launch_small_n(int prec, bool in_lds, const SmallBatchArgs &b, int n_ctx, int L_max, hipStream_t st) {
    switch (prec) {
    case kPrecC128: return launch_small_t<N, double, double>(in_lds, b, n_ctx, L_max, st);
    case kPrecC64: return launch_small_t<N, float, float>(in_lds, b, n_ctx, L_max, st);
    case kPrecC64F64: return launch_small_t<N, float, double>(in_lds, b, n_ctx, L_max, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

size_t small_lds_bytes(int N, int prec, int L, bool in_lds) {
    const int cs = prec == kPrecC128 ? 16 : 8;
    const int cc = prec == kPrecC64 ? 8 : 16;
    return small_lds_layout(N, cs, cc, L, in_lds).total;
}

size_t small_reg_lds_bytes(int L, int prec) {
    if (L < kRegMinL) return small_lds_bytes(4, prec, L, true);
    return L == 5 ? SmallReg<5>::lds : L == 6 ? SmallReg<6>::lds : SmallReg<7>::lds;
}

hipError_t launch_small_reg(int prec, const SmallBatchArgs &b, int n_ctx, hipStream_t st) {
    if (n_ctx < 1 || n_ctx > kMaxSmallBatch) return hipErrorInvalidValue;
    int threads = 0;
    size_t lds = 0;
    for (int k = 0; k < n_ctx; ++k) {
        const int L = b.c[k].L;
        if (L < 1 || L > kRegMaxL) return hipErrorInvalidValue;
        threads = std::max(threads, reg_threads(L));
        lds = std::max(lds, small_reg_lds_bytes(L, prec));
    }
    const dim3 g(n_ctx), t(threads);
    switch (prec) {
    case kPrecC128: hipLaunchKernelGGL((small_reg_kernel<double, double>), g, t, lds, st, b); break;
    case kPrecC64: hipLaunchKernelGGL((small_reg_kernel<float, float>), g, t, lds, st, b); break;
    case kPrecC64F64: hipLaunchKernelGGL((small_reg_kernel<float, double>), g, t, lds, st, b); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_small(int N, int prec, bool in_lds, const SmallBatchArgs &b, int n_ctx, int L_max,
                        hipStream_t st) {
    if (n_ctx < 1 || n_ctx > kMaxSmallBatch) return hipErrorInvalidValue;
    switch (N) {
    case 1: return launch_small_n<1>(prec, in_lds, b, n_ctx, L_max, st);
    case 4: return launch_small_n<4>(prec, in_lds, b, n_ctx, L_max, st);
    case 9: return launch_small_n<9>(prec, in_lds, b, n_ctx, L_max, st);
    case 16: return launch_small_n<16>(prec, in_lds, b, n_ctx, L_max, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace quapi
