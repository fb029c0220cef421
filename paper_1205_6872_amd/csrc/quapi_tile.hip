// Four full-window propagation steps per pass over the tensor (M = 2, N = 4),
// with the intermediate tensors kept in the registers of a block: the tile
// kernel, its tables and their launchers.
//
// Method: Dattani 2012, Sec. II (exact path-sum equation and discretized
// influence functional); the tensor-propagator step of the Introduction,
// applied up to four times per pass.
//
// A block owns a tile: the 4^4 values of the four oldest points d0..d3 times
// the 16 values of the next two digits w0, w1, 4096 entries, 16 per thread.  A
// thread holds all values of two of the points in registers, so that a step
// contracts within the thread: first (d0, d1), steps n and n+1, then, after one
// exchange through 32 KB of LDS, (d2, d3), steps n+2 and n+3.
//
// Bounds and choices (M = 2, rho at every step, one GPU, per step, before ->
// after, "before" three steps per pass in one thread's registers from L = 13 at
// complex128 and complex64/FP32 and two otherwise, with two launches for the
// rho of every step):
//   L = 15  complex128 1.18 -> 0.90 ms, complex64/FP32 0.66 -> 0.61,
//           complex64/FP64 0.93 -> 0.68.  One pass of the kept half moves
//           17.2 GB at complex128; reads and stores of the same pattern alone
//           take 3.47 ms of the 3.6 to 3.7 ms pass, so complex128 is HBM bound;
//           FP32 arithmetic is bound by its instructions: 2240 vector
//           instructions per tile and wave, 320 of them conversions (the exact FP64
//           sums of the rows that carry the trace, factors and rho terms), which
//           the vector units alone take 1.9 of the 2.4 ms for.
//   L = 13  complex64/FP64 89 -> 40 us; L = 12 complex128 57 -> 16 us; L = 10
//           28.6 -> 4.4 us; L = 8 22.4 -> 2.9 us: bound by the launch and by the
//           latency of one tile's chain; one launch per four steps, the rho of a
//           pass summed by extra blocks of the next.
//   A driven system (complex128, L = 11, rho at the last step, 64 steps): 2310 ->
//           362 us, a launch of tables and a pass per four steps where each step
//           took three launches (tables, factor products, step).
//   Calls that are not whole groups of four run parts of a pass, which move the
//   same bytes for fewer steps.  L = 15, ms per step, calls of 1 / 2 / 3 / 6 / 9:
//           complex128 3.33 / 2.79 / 1.19 / 1.19 / 1.19 -> 3.53 / 1.78 / 1.77 / 1.20 /
//           1.20; complex64/FP32 1.67 / 1.40 / 0.67 / 0.66 / 0.66 -> 1.87 / 0.94 / 0.97 /
//           0.70 / 0.73; complex64/FP64 1.76 / 0.94 / 1.20 / 0.93 / 1.02 -> 1.88 / 1.00 /
//           1.05 / 0.78 / 0.81 (three-step launches fit calls of 3, 6 and 9; a group
//           moved to where a call begins would give the call's steps other bits).
//   16 consecutive entries per store (whole cache lines): with stores of 64 B
//   from waves that run apart a pass takes 4.8 ms at L = 15; five points per
//   tile would leave 64 B stores and takes 4.8 ms for the memory alone.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "quapi_internal.h"
#include "quapi_step4.h"

namespace quapi {
namespace {

constexpr int kWaves = kBlock / 64;
constexpr int kSets = kTileSets;         // (stage, class, o in {1, 2}) factor tables

// Bits of x -> base-4 digits 3 or 0.
__device__ __forceinline__ int diagonal_digits_t(unsigned x) {
    int out = 0;
    for (int k = 0; x > 0; ++k, x >>= 1) out |= (int)(x & 1u) * 3 << (2 * k);
    return out;
}

// The high-digit value of tile index idx over k digits.  Mirror mode runs the
// values below their mirror, ordered by the place p of their highest
// off-diagonal digit (digit p is 1, those above it diagonal, those below it
// any: 2^(k-1-p) 4^p values), then the 2^k values that are their own mirror.
__device__ __forceinline__ int tile_hi(int idx, int k, bool mirror, bool *self) {
    *self = false;
    if (!mirror) return idx;
    for (int p = k - 1; p >= 0; --p) {
        const int cnt = 1 << (k - 1 + p);
        if (idx < cnt) {
            const int low = idx & ((1 << (2 * p)) - 1);
            return (diagonal_digits_t((unsigned)idx >> (2 * p)) << (2 * (p + 1))) | (1 << (2 * p)) | low;
        }
        idx -= cnt;
    }
    *self = true;
    return diagonal_digits_t((unsigned)idx);
}

// ------------------------------------------------------------------ tables
// set q = (s * 2 + cls) * 2 + (o - 1): t_w[q][w0 + 4 w1], t_u[q][u0 + 4 u1],
// t_mid[q][v], t_top[q][v], all FP64; coef as quapi_step4.h has it.
template <typename T>
__global__ void __launch_bounds__(kBlock) tile_tables_kernel(const TilePlanArgs a) {
    const BankLayout B{a.L};
    const int L = a.L;
    const int n_mid = 1 << (2 * a.d_mid), n_top = 1 << (2 * a.d_top);
    // exactly conjugate under the mirror: a pass may read an entry or its mirror,
    // and its results do not depend on which it read
    auto tab = [&](int t, int row, int col) { return tab4(a.bank, t, row, col); };
    const long long n_tab = (long long)kSets * (32 + n_mid + n_top);
    const long long total = n_tab + kTileCoefCount;
    for (long long idx = (long long)blockIdx.x * kBlock + threadIdx.x; idx < total;
         idx += (long long)gridDim.x * kBlock) {
        if (idx >= n_tab) {
            put_coef(a.coef, (int)(idx - n_tab), L, a.eta, a.s,
                     [&](int tb, int o, int p) { return a.bank[(size_t)tb * 16 + o * 4 + p]; }, sizeof(T) == 4);
            continue;
        }
        int q, v, j0, nd;
        double2 *out;
        if (idx < kSets * 16) {
            q = (int)(idx / 16); v = (int)(idx % 16); j0 = 0; nd = 2;
            out = a.t_w + idx;
        } else if (idx < kSets * 32) {
            const int k = (int)idx - kSets * 16;
            q = k / 16; v = k % 16; j0 = -1; nd = 2;
            out = a.t_u + k;
        } else if (idx < (long long)kSets * (32 + n_mid)) {
            const int k = (int)(idx - kSets * 32);
            q = k / n_mid; v = k % n_mid; j0 = 2; nd = a.d_mid;
            out = a.t_mid + k;
        } else {
            const int k = (int)(idx - (long long)kSets * (32 + n_mid));
            q = k / n_top; v = k % n_top; j0 = 2 + a.d_mid; nd = a.d_top;
            out = a.t_top + k;
        }
        const int s = q / 4, cls = q / 2 % 2, o = 1 + q % 2;
        double2 p = make_double2(1.0, 0.0);
        if (j0 == 0) {
            p = prefix4(a.bank, a.eta, a.s, L, o, cls, s % 2);       // t_w also carries these
        }
        for (int j = 0; j < nd; ++j, v >>= 2) {
            // the lag from step n+s: outer digit j0 + j; for t_u the two points
            // that are thread digits at stage s (d2, d3, then o0, o1)
            const int lag = j0 >= 0 ? L - kTileSteps - (j0 + j) + s : s < 2 ? L + s - 2 - j : s - j;
            p = cmul(p, tab(tile_tab(B, lag, cls), o, v & 3));
        }
        *out = p;
    }
}

// The parts of the tables that carry the propagator, for the group of four
// steps that starts at step n of a driven system: K of step n+s from its U, in
// the coefficients (stages 1 and 3 at lag 1, the diagonal rows of every stage),
// in t_u (stage 2: lag 1 is the thread digit o1) and, for stage 0, in the table
// t_last of the highest outer digits (lag 1 is the highest).
template <typename T>
__global__ void __launch_bounds__(kBlock) tile_drive_kernel(const TileDriveArgs a) {
    const BankLayout B{a.L};
    const int n_last = 1 << (2 * a.d_last);
    const int total = 2 * 32 + 4 * 16 + 4 * 16 + 4 * n_last;
    // K[o][p] of stage s times the influence factor at lag 1 of class cls (-1:
    // K alone), exactly conjugate under the mirror as in tile_tables_kernel
    auto kf = [&](int s, int cls, int o, int p) {
        const int k = o * 4 + p, km = mirror_d(o) * 4 + mirror_d(p);
        const int oo = km < k ? mirror_d(o) : o, pp = km < k ? mirror_d(p) : p;
        const double2 *U = a.U_t + 4 * (size_t)min(a.n + s - 1, a.n_H - 1);
        double2 v;
        if (a.k_trace_exact && oo % 3 == 0) {
            double2 col[kMaxM];
            trace_exact_column(U, 2, pp / 2, pp % 2, col);
            v = col[oo / 3];
        } else {
            const double2 u2 = U[oo % 2 * 2 + pp % 2];
            v = cmul(U[oo / 2 * 2 + pp / 2], make_double2(u2.x, -u2.y));
        }
        if (cls >= 0) v = cmul(v, a.bank[(size_t)(cls ? B.fin(1) : B.lag(1)) * 16 + oo * 4 + pp]);
        if (km < k) v.y = -v.y;
        if (km == k) v.y = 0.0;
        return v;
    };
    auto tab = [&](int t, int o, int p) { return tab4(a.bank, t, o, p); };
    for (int idx = blockIdx.x * kBlock + threadIdx.x; idx < total; idx += gridDim.x * kBlock) {
        if (idx < 64) {
            const int st = 1 + idx / 32 * 2, k = idx % 32, e = k / 8, cls = k / 4 % 2, o = 1 + k / 2 % 2;
            const double2 f = kf(st, cls, o, e);
            ((double *)a.coef)[tc_lag1(st) + k] = k % 2 ? f.y : f.x;
        } else if (idx < 128) {
            const int k = idx - 64, st = k / 16;
            const double2 f = kf(st, -1, k / 2 % 2 * 3, k / 4 % 4);
            double v = k % 2 ? f.y : f.x;
            if (sizeof(T) == 4) v = (float)v;
            ((double *)a.coef)[tc_k(0) + k] = v;
        } else if (idx < 192) {
            const int k = idx - 128, q = 8 + k / 16, v = k % 16, cls = q / 2 % 2, o = 1 + q % 2;
            a.t_u[q * 16 + v] = cmul(tab(cls ? B.fin(2) : B.lag(2), o, v & 3), kf(2, cls, o, v >> 2));
        } else {
            const int k = idx - 192, q = k / n_last, cls = q / 2, o = 1 + q % 2;
            int v = k % n_last;
            double2 p = make_double2(1.0, 0.0);
            for (int j = 0; j < a.d_last - 1; ++j, v >>= 2) {
                const int lag = a.d_last - j;
                p = cmul(p, tab(cls ? B.fin(lag) : B.lag(lag), o, v & 3));
            }
            a.t_last[k] = cmul(p, kf(0, cls, o, v));
        }
    }
}

// ---------------------------------------------------------------- exchange
// Thread layouts: A: registers (d0, d1), lane (d2, d3, w0), wave w1; B:
// registers (d2, d3), lane (w0, w1, o0), wave o1, so that a wave stores 16
// consecutive entries (whole cache lines) at a time.  Slot of an entry in the
// block's LDS: low 5 bits d2 ^ w1 | (d3 ^ (w0_hi | d0_lo << 1)) << 2 | w0_lo << 4,
// above them w1, w0_hi, d0, d1: the 8-byte accesses of 32 consecutive lanes
// cover the 64 banks once in both layouts.
struct XLane {
    int wr, rd;
    __device__ __forceinline__ XLane(int lane, int wave) {
        const int d2 = lane & 3, d3 = (lane >> 2) & 3, w = lane >> 4;
        wr = (d2 ^ wave) + ((d3 ^ (w >> 1)) << 2) + ((w & 1) << 4) + 32 * wave + 128 * (w >> 1);
        const int w0 = lane & 3, w1 = (lane >> 2) & 3, o0 = lane >> 4;
        rd = w1 + (((w0 >> 1) | (o0 & 1) << 1) << 2) + ((w0 & 1) << 4) + 32 * w1 + 128 * (w0 >> 1) + 256 * o0 +
             1024 * wave;
    }
};
// Orders this wave's LDS accesses (LDS runs a wave's accesses in order).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// The slot of register r in layouts A and B.
__device__ __forceinline__ int slot_a(const XLane &x, int r) { return (x.wr ^ ((r & 1) << 3)) + 256 * r; }
__device__ __forceinline__ int slot_b(const XLane &x, int r) { return x.rd ^ r; }
// between(): what the block does once every wave has left the buffer (and the
// phase that reads it) of the tile before.
template <typename C, typename F>
__device__ __forceinline__ void exchange(C (&w)[16], void *buf, const XLane &x, F between) {
    using X = XSlot<C>;
    typename X::type *b = (typename X::type *)buf;
#pragma unroll
    for (int part = 0; part < X::kParts; ++part) {
        __syncthreads();                   // the buffer's last readers are done
        if (part == 0) between();
#pragma unroll
        for (int r = 0; r < 16; ++r) b[slot_a(x, r)] = X::get(w[r], part);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) X::set(w[r], b[slot_b(x, r)], part);
    }
}
// ------------------------------------------------------------- rho over blocks
// rho of one step from its block rows (4 complex values each), compensated,
// in a fixed order: a thread takes one of the 8 doubles of every 32nd row,
// the 32 row lanes are combined in a wave and then over the waves.
__device__ void tile_rho_sum(const double *__restrict__ rows, int n_rows, double *out, double2 *s_x) {
    const int t = threadIdx.x, q = t & 7, lane = t & 63, wave = t >> 6;
    double s = 0.0, c = 0.0;
    int r = t >> 3;
    constexpr int U = 4, kStep = kBlock / 8;
    for (; r + (U - 1) * kStep < n_rows; r += U * kStep) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = rows[(size_t)(r + u * kStep) * 8 + q];
#pragma unroll
        for (int u = 0; u < U; ++u) neumaier(s, c, v[u]);
    }
    for (; r < n_rows; r += kStep) neumaier(s, c, rows[(size_t)r * 8 + q]);
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) {
        const double s2 = __shfl_xor(s, off, 64), c2 = __shfl_xor(c, off, 64);
        // the lower lane's pair first on both sides, so that both hold the same
        double a = (lane & off) ? s2 : s, ac = (lane & off) ? c2 : c;
        two_sum_combine(a, ac, (lane & off) ? s : s2, (lane & off) ? c : c2);
        s = a;
        c = ac;
    }
    if (lane < 8) s_x[wave * 8 + lane] = make_double2(s, c);
    __syncthreads();
    if (t < 8) {
        double2 a = s_x[t];
        for (int w = 1; w < kWaves; ++w) two_sum_combine(a.x, a.y, s_x[w * 8 + t].x, s_x[w * 8 + t].y);
        out[t] = a.x + a.y;
    }
}

__global__ void __launch_bounds__(kBlock) tile_rho_kernel(const TileRho r) {
    __shared__ double2 s_x[kWaves * 8];
    tile_rho_sum((const double *)r.rows[blockIdx.x], r.n_rows, (double *)r.out[blockIdx.x], s_x);
}

// --------------------------------------------------------------------- pass
// Stages s0 .. s1-1 of the group of four steps n .. n+3 (n > L, n - L - 1 a
// multiple of 4).  The stage range only says which of the steps run and where
// the entries are read and written: every entry and every rho sum is formed
// by the same operations whatever the ranges a group is run in.
// PART: kWhole all four stages; kFront some of stages 0 and 1 (no exchange);
// kBack any other range (one kernel for all of them holds more registers than
// there are: M = 2, L = 15, complex128, 3.70 -> 4.18 ms a whole pass).  S0: the
// first stage, which decides where a register's entry lies; in a tile below its
// mirror that also says which entries are read or stored at their mirror, so
// that their addresses are two bases plus uniform offsets (mirrored entry by
// entry in 64 bits -> this, L = 15, rho at every step: stages 0 to 2 complex128
// 4.06 -> 3.52 ms, complex64/FP32 2.79 -> 2.12; stage 0 3.45 -> 3.38, 2.06 -> 1.73).
// AHEAD (FP64 arithmetic): a tile is read after the first stage of the tile
// before it, which frees the registers; with the reads in flight under the
// other stages and ahead of the stores two waves per SIMD do better than three
// without them (L = 15, complex128, 3.90 -> 3.66 ms a pass, against 3.47 ms for
// the reads and stores alone), but only where a block has several tiles.
enum { kWhole, kFront, kBack };
template <typename S, typename T, bool RHO, bool MIRROR, int PART, int S0, bool AHEAD>
__global__ void __launch_bounds__(kBlock, AHEAD ? 2 : 3) tile_kernel(const TileArgs a) {
    constexpr bool WHOLE = PART == kWhole;
    static_assert(S0 == 0 || !WHOLE, "a whole pass begins at stage 0");
    using C = typename Cx<T>::type;
    using CS = typename Cx<S>::type;
    __shared__ __align__(16) unsigned char s_buf[kWaves][1024 * 8];
    __shared__ double2 s_u[kSets * 16];
    __shared__ double2 s_w[kWaves][64];              // [w1][set][w0]
    double2 *const s_red = (double2 *)s_buf;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    if ((int)blockIdx.x >= a.n_work) {
        // the rho of the pass before (its rows were written by another launch)
        const int k = (int)blockIdx.x - a.n_work;
        tile_rho_sum((const double *)a.prev.rows[k], a.prev.n_rows, (double *)a.prev.out[k], s_red);
        return;
    }
    // Block of the pass.  Parts at complex128 give neighbouring blocks, whose tiles
    // are neighbours in memory, to one XCD (L = 15, stages 2 and 3 3.98 -> 3.65 ms,
    // stages 0 and 1 3.63 -> 3.45; a whole pass 3.70 -> 3.72 and complex64 parts
    // 1.79 -> 1.83 ms the other way: they keep the order of the launch)
    const int blk = PART != kWhole && sizeof(S) == 8 && a.n_work % 8 == 0
                        ? (int)(blockIdx.x & 7) * (a.n_work >> 3) + (int)(blockIdx.x >> 3)
                        : (int)blockIdx.x;
    const T *coef = (const T *)a.coef;
    // layout A: lane (d2, d3, w0); layout B: lane (w0, o0, o1); w1 = wave
    double acc[RHO ? kTileSteps : 1][MIRROR ? 1 : 2];
#pragma unroll
    for (int s = 0; s < (RHO ? kTileSteps : 1); ++s)
#pragma unroll
        for (int k = 0; k < (MIRROR ? 1 : 2); ++k) acc[s][k] = 0.0;
    const int s1 = a.s1;
    const CS *__restrict__ ain = (const CS *)a.a_in;
    CS *__restrict__ aout = (CS *)a.a_out;
    const long long mc = a.m_count;

    // The entries of a tile, with the tile's table values.
    CS x[16];                              // as stored (converting waits for the read)
    double2 top, mid;
    const double2 tw = a.t_w[(lane >> 2) * 16 + (lane & 3) + 4 * wave];
    // Part of a group: the index of the thread's entry of registers zero, in layout
    // A or, for stage 3 alone, in layout B, which stage 3 works in (no exchange:
    // L = 15, complex64 2.21 -> 1.99 ms; stages 2 and 3 read in it 1.99 -> 2.20).
    // The points of the group's earlier stages, in the place of d0, d1, d2, are
    // the highest digits, and the tile's come next: registers' digits planes
    // apart, and after stages 0 and 2 the lowest digit in memory.
    auto part_in = [&](int hi, int lane) {
        const int wl = lane & 15, ul = (lane >> 4) + 4 * wave;
        if (S0 < 3) return ((long long)hi * 16 + ul) * (S0 == 1 ? 64 : 16) + (S0 == 1 ? 4 : 1) * wl;
        return ((long long)hi * 16 + wl) * 4 + (ul & 3) * (mc << 2) + (ul >> 2) * (mc << 4);
    };
    auto part_reg = [&](int r) {
        return S0 == 2 ? (r & 3) * (mc << 4) + (r >> 2) * (mc << 6) : (r & 3) * (mc << 6) + (r >> 2);
    };
    // stage 3: whether the lane's digits put its entries below their mirror, for
    // the registers whose own highest digit leaves it open
    auto lane_direct = [&](int lane) {
        const int ul = (lane >> 4) + 4 * wave;
        return !MIRROR || ul <= mirror_d(ul & 3) + 4 * mirror_d(ul >> 2);
    };
    auto by_lane = [](int r) { return MIRROR && S0 == 3 && ((r & 3) == 0 || (r & 3) == 3); };
    constexpr bool kSwap = sizeof(S) == 4;
    auto read_tile = [&](int hi, bool self, int lane) {
        const int set = lane >> 2, ua = lane & 15, wa = lane >> 4;
        top = a.t_top[((size_t)set << (2 * a.d_top)) + (hi >> (2 * a.d_mid))];
        mid = a.t_mid[((size_t)set << (2 * a.d_mid)) + (hi & ((1 << (2 * a.d_mid)) - 1))];
        if constexpr (S0 == 0) {
            // a tile that is its own mirror: the entries above their mirror hold
            // no valid value, their mirror's conjugate (of the same tile) does
            const int b = (wa + 4 * wave) * 256 + 16 * ua, bm = MIRROR ? (int)mirror4(b) : b;
            const CS *p = ain + (long long)hi * 4096 + (self ? min(b, bm) : b);
            if (!self) {
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = p[r];
                // the reads of each branch stay whole and in it (merged over the
                // branches they are split into components: 3.7 -> 4.6 ms a pass)
                asm volatile("" ::: "memory");
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int rm = (int)mirror4(r);
                    x[r] = p[b < bm ? r : b > bm ? rm : min(r, rm)];
                }
                asm volatile("" ::: "memory");
            }
        } else {
            // a part: an entry above its mirror through the mirror.  In a tile below
            // its mirror complex64 reads whole runs of the registers' lowest digit
            // (stages 1 to 3 entry by entry 2.23 -> 2.03 ms; stage 1 alone, which has
            // the time, 1.79 -> 1.83: entry by entry); where that is at the mirror
            // for some lanes only, fix_tile puts them in order
            const long long x0 = part_in(hi, lane), x0m = MIRROR ? mirror4(x0) : x0;
            if (!self) {
                const CS *const pd = ain + x0, *const pm = ain + x0m, *const pl = lane_direct(lane) ? pd : pm;
                if constexpr (S0 == 2) {
                    long long da = mc << 4, db = mc << 6;
                    asm volatile("" : "+s"(da), "+s"(db));     // their multiples are not kept over the tiles
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int rm = (int)mirror4(r), rr = MIRROR && rm < r ? rm : r;
                        x[r] = (MIRROR && rm < r ? pm : pd)[(rr & 3) * da + (rr >> 2) * db];
                        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
                    long long one = 1;
                    if (PART == kFront) asm volatile("" : "+s"(one));
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const bool flip = MIRROR && g == 2;
                        const CS *const q = (flip ? pm : S0 == 1 || g == 1 ? pd : pl) + (flip ? 1 : g) * (mc << 6);
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            x[g + 4 * c] = q[(flip ? mirror_d(c) : kSwap || !by_lane(g) || lane_direct(lane) ? c : mirror_d(c)) * one];
                    }
                }
                asm volatile("" ::: "memory");
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const long long i = x0 + part_reg(r), im = x0m + part_reg((int)mirror4(r));
                    x[r] = ain[im < i ? im : i];
                    if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
                asm volatile("" ::: "memory");
            }
        }
    };
    // the conjugates of the entries that were read at their mirror
    auto fix_tile = [&](int hi, bool self, int lane) {
        if (!MIRROR || (S0 == 0 && !self)) return;
        const int ua = lane & 15, wa = lane >> 4;
        if (!self) {
            const bool d = lane_direct(lane);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (S0 == 2 ? (int)mirror4(r) < r : S0 > 0 && (r & 3) == 2) x[r].y = -x[r].y;
                const int rm = (r & 3) + 4 * mirror_d(r >> 2);
                if (!by_lane(r) || rm < r) continue;
                const CS u = x[r], um = x[rm];
                const CS v = kSwap ? um : u, vm = kSwap ? u : um;
                x[r].x = d ? u.x : v.x;
                x[r].y = d ? u.y : -v.y;
                if (rm == r) continue;
                x[rm].x = d ? um.x : vm.x;
                x[rm].y = d ? um.y : -vm.y;
            }
            return;
        }
        const long long x0 = S0 == 0 ? (wa + 4 * wave) * 256 + 16 * ua : part_in(hi, lane);
        const long long x0m = mirror4(x0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int rm = (int)mirror4(r);
            const long long i = x0 + (S0 == 0 ? r : part_reg(r)), im = x0m + (S0 == 0 ? rm : part_reg(rm));
            if (im < i) x[r].y = -x[r].y;
            if (im == i) x[r].y = 0.0f;              // its own conjugate (another kernel's rounding aside)
        }
    };
    const int k_hi = a.d_mid + a.d_top;
    bool self, self_next = false;
    int hi = tile_hi(blk, k_hi, MIRROR, &self), hi_next = 0;
    if (AHEAD) read_tile(hi, self, lane);
    for (int idx = blk; idx < a.n_tiles; idx += a.n_work, hi = hi_next, self = self_next) {
        // opaque per tile: what the lane's position gives (LDS slots, offsets)
        // is formed again for each tile rather than held in registers
        int lane = t & 63;
        asm volatile("" : "+v"(lane));
        const XLane xl(lane, wave);
        const int ua = lane & 15, wa = lane >> 4;
        const int wb = lane & 15, ub = (lane >> 4) + 4 * wave;
        C w[16];
        if (!AHEAD) read_tile(hi, self, lane);
        if (idx == blk) {
            s_u[t] = a.t_u[t];         // once, behind the first tile's loads
            __syncthreads();
        }
        // lane set * 4 + w0 forms the factor of its set for the wave's w1.  The
        // sets of stages 0 and 1 (lanes 0 .. 31) are read by this wave only;
        // those of stages 2 and 3 by every wave, after the exchange's barriers
        double2 tile_f;
        {
            tile_f = cmul(cmul(top, mid), tw);
            wave_fence();
            if (S0 < 2 && lane < 32) s_w[wave][lane] = tile_f;
            wave_fence();
        }
        // the factor of set q over the thread's fixed digits, w0 + 4 w1 = wl
        auto factor = [&](int q, int wl, int ul) {
            return cmul(s_w[wl >> 2][q * 4 + (wl & 3)], s_u[q * 16 + ul]);
        };
        const int wl = wa + 4 * wave;
        // one stage's rho terms into the running sums
        auto add_rho = [&](int s, int wl, int ul, double2 tf1, double2 tf2, double2 v0, double2 v3) {
            const double2 v1 = cmul(factor(4 * s + 2, wl, ul), tf1);
            const double2 v2 = cmul(factor(4 * s + 3, wl, ul), tf2);
            if constexpr (MIRROR) {
                // a tile below its mirror also stands for the mirrored tile
                // (conjugate, points 1 and 2 swapped); rho[2] = conj(rho[1])
                const double two = self ? 1.0 : 2.0, one = self ? 0.0 : 1.0;
                acc[s][0] = row_add(acc[s][0], two * v0.x, 0, lane);
                acc[s][0] = row_add(acc[s][0], two * v3.x, 1, lane);
                acc[s][0] = row_add(acc[s][0], fma(one, v2.x, v1.x), 2, lane);
                acc[s][0] = row_add(acc[s][0], fma(-one, v2.y, v1.y), 3, lane);
            } else {
                acc[s][0] = row_add(acc[s][0], v0.x, 0, lane);
                acc[s][0] = row_add(acc[s][0], v0.y, 1, lane);
                acc[s][0] = row_add(acc[s][0], v1.x, 2, lane);
                acc[s][0] = row_add(acc[s][0], v1.y, 3, lane);
                acc[s][1] = row_add(acc[s][1], v2.x, 0, lane);
                acc[s][1] = row_add(acc[s][1], v2.y, 1, lane);
                acc[s][1] = row_add(acc[s][1], v3.x, 2, lane);
                acc[s][1] = row_add(acc[s][1], v3.y, 3, lane);
            }
        };
        double2 tf1, tf2, rd0, rd3;
        // storage narrower than the arithmetic: the values are rounded to it where
        // a call may end without changing the result, after the pairs (n, n+1)
        // and (n+2, n+3), or for a driven system after every step
        auto round_to_storage = [&](bool on) {
            if (sizeof(S) < sizeof(T) && on) {
#pragma unroll
                for (int r = 0; r < 16; ++r) w[r] = conv<C>(conv<CS>(w[r]));
            }
        };
        fix_tile(hi, self, lane);
        // (a.s0 is S0: the branch keeps the stage's registers apart from the read's,
        // 119 instead of 136 of them in a whole pass of FP32 arithmetic)
        if (S0 == 0 && a.s0 <= 0) {
            const int prev = hi >> (2 * (k_hi - 1));                   // point n-1
            double2 k0, k3;
            coef_k(coef, 0, prev, k0, k3);
            tile_stage<T, RHO, MIRROR, 0>(x, w, coef, factor(0, wl, ua), factor(1, wl, ua), k0, k3, tf1, tf2, rd0,
                                          rd3);
            if (RHO) add_rho(0, wl, ua, tf1, tf2, rd0, rd3);
            round_to_storage(a.round_each);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) w[r] = conv<C>(x[r]);
        }
        if (idx + a.n_work < a.n_tiles) {
            hi_next = tile_hi(idx + a.n_work, k_hi, MIRROR, &self_next);
            if (AHEAD) read_tile(hi_next, self_next, lane);
        }
        if (S0 <= 1 && s1 > 1) {
            tile_stage<T, RHO, MIRROR, 1>(w, w, coef, factor(4, wl, ua), factor(5, wl, ua), double2{}, double2{}, tf1, tf2, rd0, rd3);
            if (RHO) add_rho(RHO ? 1 : 0, wl, ua, tf1, tf2, rd0, rd3);
            round_to_storage(true);
        }
        // the 16 entries y0 + (r % 4) da + (r / 4) db of a part of a group: in a tile
        // below its mirror at the mirrored address, conjugated, unless direct(r); a
        // tile that is its own mirror stores only those not above it
        auto store_part = [&](long long y0, long long da, long long db, auto direct) {
            asm volatile("" : "+s"(da), "+s"(db));     // their multiples are not kept over the tiles
            const long long y0m = MIRROR ? mirror4(y0) : y0;
            if (!self) {
                CS *const pd = aout + y0, *const pm = aout + y0m;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int rm = (int)mirror4(r);
                    const long long off = (r & 3) * da + (r >> 2) * db, offm = (rm & 3) * da + (rm >> 2) * db;
                    const bool dir = !MIRROR || direct(r, rm);
                    C v = w[r];
                    if (!dir) v.y = -v.y;
                    *(dir ? pd + off : pm + offm) = conv<CS>(v);
                    if (r % 2 == 1) __builtin_amdgcn_sched_barrier(0);
                }
                return;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rm = (int)mirror4(r);
                const long long y = y0 + (r & 3) * da + (r >> 2) * db;
                const long long ym = y0m + (rm & 3) * da + (rm >> 2) * db;
                if (!(ym < y)) aout[y] = conv<CS>(w[r]);
                if (r % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
        };
        // lane digits (A, B, C), register digit q = r / 4 -> lane (q, A, C),
        // register B, through the wave's part of the buffer: after an odd number
        // of stages the lowest digit in memory is a register's (stored from
        // there, 16 B of a lane at a time, M = 2, L = 15, complex128: stage 0
        // alone 4.74 -> 3.48 ms, stage 2 alone 6.26 -> 3.88, stages 0 to 2 4.73
        // -> 4.09)
        auto rotate = [&]() {
            C *const b = (C *)s_buf[wave];
            const int A = lane & 3, B = (lane >> 2) & 3, c6 = (lane >> 4) << 6;
#pragma unroll
            for (int ra = 0; ra < 4; ++ra) {
                wave_fence();
#pragma unroll
                for (int q = 0; q < 4; ++q) b[(q ^ B) + (A << 2) + (B << 4) + c6] = w[ra + 4 * q];
                wave_fence();
#pragma unroll
                for (int q = 0; q < 4; ++q) w[ra + 4 * q] = b[(A ^ q) + (B << 2) + (q << 4) + c6];
            }
        };
        if constexpr (PART == kFront) {
            // the digits that follow each other in memory are the lane's: d2, d3,
            // w0 after stage 1, and d1, d2 after stage 0
            // (the highest digits of an output are o0, or o1 and o0, in the registers)
            const long long m = (long long)hi * 16 + 4 * wave + wa;
            if (S0 == 0 && s1 == 1) {
                rotate();
                store_part(m * a.out_m + (ua & 3) * a.out_d[1] + (ua >> 2) * a.out_d[2], a.out_d[0], a.out_d[3],
                           [](int r, int) { return (r & 3) != 2; });
            } else {
                store_part(m * a.out_m + (ua & 3) * a.out_d[2] + (ua >> 2) * a.out_d[3], a.out_d[0], a.out_d[1],
                           [](int r, int rm) { return r <= rm; });
            }
        } else {
        if constexpr (S0 < 3) {
            exchange(w, s_buf, xl, [&]() {
                if (lane >= 32) s_w[wave][lane] = tile_f;
            });
        } else {                           // read in layout B
            __syncthreads();               // the factors' last readers (of the tile before) are done
            if (lane >= 32) s_w[wave][lane] = tile_f;
            __syncthreads();
        }
        if (S0 <= 2 && s1 > 2) {
            double2 k0, k3;
            coef_k(coef, 2, wave, k0, k3);
            tile_stage<T, RHO, MIRROR, 2>(w, w, coef, factor(8, wb, ub), factor(9, wb, ub), k0, k3, tf1, tf2, rd0, rd3);
            if (RHO) add_rho(RHO ? 2 : 0, wb, ub, tf1, tf2, rd0, rd3);
            round_to_storage(a.round_each);
        }
        if (s1 > 3) {
            tile_stage<T, RHO, MIRROR, 3>(w, w, coef, factor(12, wb, ub), factor(13, wb, ub), double2{}, double2{}, tf1, tf2, rd0, rd3);
            if (RHO) add_rho(RHO ? 3 : 0, wb, ub, tf1, tf2, rd0, rd3);
        }
        const long long m = (long long)hi * 16 + wb;        // layout B's m
        const int ubm = mirror_d(ub & 3) + 4 * mirror_d(ub >> 2);
        if (WHOLE) {
            // an output above its mirror goes to the mirrored address as its
            // conjugate (the entry the mirrored tile, which does not run, owns);
            // a tile that is its own mirror forms those entries too, and stores
            // only the ones not above their mirror
            CS *const pd = aout + m + mc * ub;
            CS *const pm = aout + mirror4(m) + mc * ubm;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rm = (int)mirror4(r);
                const bool direct = !MIRROR || r < rm || (r == rm && ub <= ubm);
                if (MIRROR && self && (!direct || (r == rm && ub == ubm && wb > (int)mirror4(wb)))) continue;
                C v = w[r];
                if (!direct) v.y = -v.y;
                // the 16 plane offsets are formed per store, not all kept
                long long plane = 16 * mc;
                asm volatile("" : "+s"(plane));
                CS *const p = (direct ? pd : pm) + plane * (direct ? r : rm);
                *p = conv<CS>(v);
            }
        } else if (s1 == 3) {
            __syncthreads();                       // every wave has read its exchanged entries
            rotate();                              // lane (d3, w0, o0), registers (o2, w1)
            store_part(((long long)hi * 16 + (wb >> 2)) * a.out_m + (wb & 3) * a.out_d[3] +
                           (ub & 3) * a.out_d[0] + (ub >> 2) * a.out_d[1],
                       a.out_d[2], 4 * a.out_m,
                       [&](int r, int) { return (r & 3) == 1 || ((r & 3) != 2 && ub <= ubm); });
        } else {
            store_part(m * a.out_m + (ub & 3) * a.out_d[0] + (ub >> 2) * a.out_d[1], a.out_d[2], a.out_d[3],
                       [&](int r, int rm) { return r < rm || (r == rm && ub <= ubm); });
        }
        }
    }
    if constexpr (RHO) {
        // rows of the block: [stage][block][4 complex]
        __syncthreads();                   // s_red shares the exchange buffer
#pragma unroll
        for (int s = 0; s < kTileSteps; ++s) {
#pragma unroll
            for (int k = 0; k < (MIRROR ? 1 : 2); ++k) {
                double v = acc[s][k];
                for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
                if ((lane & 15) == 0) ((double *)s_red)[((s * 2 + k) * kWaves + wave) * 4 + (lane >> 4)] = v;
            }
        }
        __syncthreads();
        if (t < kTileSteps * 8) {
            const int s = t / 8, q = t % 8;    // double q of the row: (rho[q / 2]).(q % 2)
            auto sum = [&](int k, int row) {
                double v = 0.0;
                for (int w = 0; w < kWaves; ++w) v += ((const double *)s_red)[((s * 2 + k) * kWaves + w) * 4 + row];
                return v;
            };
            double v;
            if (MIRROR) v = q == 0 ? sum(0, 0) : q == 6 ? sum(0, 1) : q == 2 || q == 4 ? sum(0, 2)
                          : q == 3 ? sum(0, 3) : q == 5 ? -sum(0, 3) : 0.0;
            else v = sum(q / 4, q % 4);
            ((double *)a.rows)[((size_t)s * a.n_work + blk) * 8 + q] = v;
        }
    }
}

template <typename S, typename T, bool RHO, bool MIRROR, bool AHEAD>
hipError_t launch_tile_w(const TileArgs &a, hipStream_t st) {
    const dim3 g(a.n_work + a.prev.n), b(kBlock);
    if (a.s0 < 0 || a.s0 >= a.s1 || a.s1 > kTileSteps) return hipErrorInvalidValue;
#define QUAPI_TILE(PART, S0) hipLaunchKernelGGL((tile_kernel<S, T, RHO, MIRROR, PART, S0, AHEAD>), g, b, 0, st, a)
    if (a.s1 - a.s0 == kTileSteps) QUAPI_TILE(kWhole, 0);
    else if (a.s1 <= 2 && a.s0 == 0) QUAPI_TILE(kFront, 0);
    else if (a.s1 <= 2) QUAPI_TILE(kFront, 1);
    else if (a.s0 == 0) QUAPI_TILE(kBack, 0);
    else if (a.s0 == 1) QUAPI_TILE(kBack, 1);
    else if (a.s0 == 2) QUAPI_TILE(kBack, 2);
    else QUAPI_TILE(kBack, 3);
#undef QUAPI_TILE
    return hipGetLastError();
}
template <typename S, typename T>
hipError_t launch_tile_t(bool rho, bool mirror, const TileArgs &a, hipStream_t st) {
    // Tiles are read ahead from eight per block (mirror mode: L = 13) on: with
    // two or three a block finishes sooner three to a compute unit (L = 12,
    // complex128, 60 steps: 1.06 ms ahead, 1.02 ms not).  FP32 arithmetic fits
    // four waves per SIMD and is bound by its instructions either way.
    if constexpr (sizeof(T) == 8) {
        if (mirror && a.n_tiles >= 8 * a.n_work)
            return rho ? launch_tile_w<S, T, true, true, true>(a, st) : launch_tile_w<S, T, false, true, true>(a, st);
    }
    if (rho)
        return mirror ? launch_tile_w<S, T, true, true, false>(a, st) : launch_tile_w<S, T, true, false, false>(a, st);
    return mirror ? launch_tile_w<S, T, false, true, false>(a, st) : launch_tile_w<S, T, false, false, false>(a, st);
}

}  // namespace

hipError_t launch_tile(int prec, bool rho, bool mirror, const TileArgs &a, hipStream_t st) {
    switch (prec) {
    case kPrecC128: return launch_tile_t<double, double>(rho, mirror, a, st);
    case kPrecC64: return launch_tile_t<float, float>(rho, mirror, a, st);
    case kPrecC64F64: return launch_tile_t<float, double>(rho, mirror, a, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_tile_rho(const TileRho &r, hipStream_t st) {
    if (r.n < 1) return hipSuccess;
    hipLaunchKernelGGL(tile_rho_kernel, dim3(r.n), dim3(kBlock), 0, st, r);
    return hipGetLastError();
}

hipError_t launch_tile_tables(int prec, const TilePlanArgs &a, hipStream_t st) {
    const long long total =
        (long long)kSets * (32 + (1LL << (2 * a.d_mid)) + (1LL << (2 * a.d_top))) + kTileCoefCount;
    const dim3 g((unsigned)std::min<long long>(1024, (total + kBlock - 1) / kBlock)), b(kBlock);
    if (prec == kPrecC64) hipLaunchKernelGGL(tile_tables_kernel<float>, g, b, 0, st, a);
    else hipLaunchKernelGGL(tile_tables_kernel<double>, g, b, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_tile_drive(int prec, const TileDriveArgs &a, hipStream_t st) {
    const int total = 2 * 32 + 8 * 16 + (4 << (2 * a.d_last));
    const dim3 g((total + kBlock - 1) / kBlock), b(kBlock);
    if (prec == kPrecC64) hipLaunchKernelGGL(tile_drive_kernel<float>, g, b, 0, st, a);
    else hipLaunchKernelGGL(tile_drive_kernel<double>, g, b, 0, st, a);
    return hipGetLastError();
}

}  // namespace quapi
