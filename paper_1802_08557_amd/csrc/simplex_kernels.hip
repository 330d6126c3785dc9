// simplex_kernels.hip -- the batched dense-tableau simplex for gfx950.
//
// One workgroup solves one LP at a time and pops the next LP from a work
// counter (a persistent launch sized to what the device holds at once).  The
// paper maps one CUDA block to one LP (Sec. 5.1, load balancing) and uses the
// block's threads inside the tableau; here a workgroup of NT threads (one or
// more 64-wide wavefronts) does the same, with the tableau kept in LDS when it
// fits the launch's LDS budget and in an HBM scratch slot of the workgroup
// otherwise.
//
// The tableau is the condensed ("exchange") form of the paper's Sec. 4.1
// tableau: the m basic columns are unit vectors and are not stored, so a row
// holds the N non-basic columns, and a pivot swaps the entering and leaving
// variables' columns in place.  The right-hand sides, the reduced costs
// (entering candidates have d_j > 0) and minus the objective value are kept
// beside it, always current.  basis[i] / nonb[j] hold the Bland index of the
// variable of row i / column j.
//
// Per iteration (Sec. 4.1):
//   Step 1 (pricing): argmax of d_j > eps_opt over eligible columns, ties to
//     the smallest Bland index; Bland's smallest-index rule after k_deg
//     consecutive degenerate pivots, until a pivot makes progress.
//   Step 2 (ratio): argmin of max(b_i, 0) / a_ie over rows with a_ie > tol_piv,
//     ties to the smallest Bland index of the basic variable; none: unbounded.
//     Wavefront DPP reductions and ballots on (key, Bland index), then one
//     slot per wavefront in LDS, stand in for the paper's Data[]/Indices[]
//     arrays.
//   Step 3 (pivot): pivot row / PE; every other row (objective included) minus
//     a_ie times the new pivot row (Listing 1); the entering column becomes the
//     leaving variable's column: 1/PE in the pivot row, -a_ie/PE elsewhere.
//     Every element takes one fma per pivot, the same expression wherever the
//     tableau lives, so results do not depend on the placement or the
//     workgroup size.  The updates of up to 32 pivots wait in a window of
//     vectors and reach the tableau in one sweep on the matrix cores (flush).
// Phase I (Sec. 4) maximises -(sum of artificials) when some row needs one;
// basic artificials at zero are driven out and redundant rows dropped, then
// Phase II prices c out over the basis and continues.
#include <math.h>

#include "device_common.h"
#include "internal.h"

namespace lpb {
namespace {

constexpr int LE = 0, GE = 1, EQ = 2;
constexpr int ST_OPTIMAL = 0, ST_INFEASIBLE = 1, ST_UNBOUNDED = 2, ST_ITER = 3,
              ST_NUMERICAL = 4, ST_INVALID = 5;
constexpr int BIG = 0x7fffffff;
constexpr int ROW_NEG = 1, ROW_DEAD = 8;

template <typename T>
struct Ctrl {
    int ng, nart, neq, bad;
    int next;
    int cnt;  // scratch tally (warm start)
    int inf;  // overflowed: an infinity or NaN was seen
    int pad;
    T rv[2][8];  // block_pick: one slot per wavefront, two sets used in turn
    int ri[2][8];
    int rp[2][8];
    double rd[16];
};

__device__ __forceinline__ int row_sense(int f) { return (f >> 1) & 3; }

// ---- reductions ------------------------------------------------------------

// The workgroup's largest of values >= +0 (not NaN).
template <typename T, int NT>
__device__ __forceinline__ double block_max(double v, Ctrl<T> *sh)
{
    v = lane_get(v, __builtin_ctzll(wave_max_nonneg(true, v)));
    if constexpr (NT > 64) {
        const int w = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) sh->rd[w] = v;
        __syncthreads();
        v = sh->rd[0];
#pragma unroll
        for (int q = 1; q < NT / 64; ++q) v = fmax(v, sh->rd[q]);
        __syncthreads();
    }
    return v;
}

// The lane of the wavefront with the largest (MAX) or least value among `on`
// lanes, ties to the smallest `tie`; -1 when no lane is on.  Values are >= +0
// and not NaN.
template <bool MAX, typename T>
__device__ __forceinline__ int wave_pick(bool on, T v, int tie)
{
    uint64_t mask = MAX ? wave_max_nonneg(on, v) : wave_min_nonneg(on, v);
    if (!mask) return -1;
    if (__builtin_expect(__popcll(mask) > 1, 0)) {
        const bool in = (mask >> (threadIdx.x & 63)) & 1;
        const int least = wave_min_i(in ? tie : BIG);
        mask = ballot(in && tie == least);
    }
    return __builtin_ctzll(mask);
}

// A thread's own best candidate over the items it looks at.
template <bool MAX, typename T>
struct Best {
    bool on = false;
    T v = T(0);
    int tie = BIG, idx = -1;
    __device__ __forceinline__ void offer(bool ok, T x, int t, int i)
    {
        const bool take = ok && (!on || (MAX ? x > v : x < v) || (x == v && t < tie));
        v = take ? x : v;
        tie = take ? t : tie;
        idx = take ? i : idx;
        on |= ok;
    }
};

// ---- one LP ------------------------------------------------------------------

template <typename T, int NT>
struct LP {
    // geometry
    int m, n, N, ld, nart;
    int64_t k, ro, co;
    const double *A, *b, *c;
    const int32_t *rows;  // screened LP: row i is constraint rows[i] of the shared LP
    int m_full;
    // Constraint of the (shared) LP that row i reads, clamped into range.
    __device__ __forceinline__ int row_of(int i) const
    {
        if (!rows) return i;
        const int q = rows[i];
        return (q >= 0 && q < m_full) ? q : 0;
    }
    // LDS arrays
    Ctrl<T> *sh;
    int *basis, *nonb, *rowf, *colrow;
    T *rhs, *obj;  // current right-hand sides and reduced costs
    T *np, *pr;    // window: negated pivot columns [K][m], scaled pivot rows [K][N]
    int K, p;      // pivots the window holds at most, and now
    bool direct;   // each pivot updates the tableau at once; the window stays empty
    bool steep;    // steepest-edge pricing
    T *tab;        // m x N in LDS or device memory, row stride ld, without the window's pivots
    T z;           // right-hand side of the objective row (minus its value)
    int turn;      // set of block_pick's slots
    // counters (uniform across the workgroup)
    int iters, it1, degp, cap;
};

// The workgroup's best candidate (see wave_pick): its idx and, in `best`, its
// value; -1 when there is none.  One barrier: the slots of consecutive calls
// alternate.
template <bool MAX, typename T, int NT>
__device__ __forceinline__ int block_pick(LP<T, NT> &P, const Best<MAX, T> &c, T &best)
{
    const int lane = threadIdx.x & 63;
    int src = wave_pick<MAX>(c.on, c.v, c.tie);
    if constexpr (NT == 64) {
        if (src < 0) return -1;
        best = lane_get(c.v, src);
        return lane_get(c.idx, src);
    } else {
        Ctrl<T> *sh = P.sh;
        const int w = uniform(threadIdx.x >> 6), t = P.turn;
        P.turn ^= 1;
        if (lane == max(src, 0)) {
            sh->rv[t][w] = c.v;
            sh->ri[t][w] = c.tie;
            sh->rp[t][w] = src < 0 ? -1 : c.idx;
        }
        __syncthreads();
        const int q = lane & (NT / 64 - 1);
        const T v = sh->rv[t][q];
        const int tie = sh->ri[t][q], idx = sh->rp[t][q];
        src = wave_pick<MAX>(lane < NT / 64 && idx >= 0, v, tie);
        if (src < 0) return -1;
        best = lane_get(v, src);
        return lane_get(idx, src);
    }
}

// The current tableau is
//     t_ij = fma(np[p-1]_i, pr[p-1]_j, ... fma(np[0]_i, pr[0]_j, tab_ij) ...)
// over the pivots of the window, oldest first.  A pivot's own row and column,
// which it replaces rather than updates, go to tab at once and the window's
// entries of that row and column become 0 (push), so that every entry takes
// the operations of one sweep per pivot in their order, and the sweep (flush)
// comes once per K pivots.  (Past the range of T the two differ: 0 times infinity
// leaves NaN in an entry that its pivot replaced.  See overflowed.)
//
// Why a window: the sweep reads and writes the whole tableau, which for the
// large LPs of a batch lives in device memory and bounds the kernel by the
// rate of the memory behind the CU, while Steps 1 and 2 need the reduced costs
// and right-hand sides (kept current in LDS), one column and one row.  K is
// what the LP's LDS leaves (LdsLayout), at most kMaxWindow.  Measured against
// three pivots per sweep on the vector units: 1,000 LPs of 500 x 500 FP64 23.5 ->
// 7.3 ms (sixteen pivots per sweep), 10,000 uneven LPs of 10..300 FP64 140 -> 59 ms
// and FP32 86 -> 41 ms, 2,000 LPs of 117 x 150 FP32 1.14 -> 0.55 ms.
//
// A tableau in LDS is swept at LDS speed, so sixteen pivots a window do: each pivot
// reads half as many vectors of it as of thirty-two (1,000 LPs FP64, 32 / 16 pivots:
// 100 x 100 344 / 335 us, 200 x 60 FP32 322 / 316 us).  Of at most kDirectRows rows
// each pivot updates every entry at once (push), a few operations a column against
// walks over the window for the column and the row: 1,000 LPs FP64 of 3 x 500 98 ->
// 77 us, of 10 x 91 94 -> 84 us, of 16 x 100 93 -> 92 us, of 24 x 70 100 -> 107 us,
// hence the line at twelve.
constexpr int kMaxWindow = 32;
constexpr int kMaxWindowLds = 16;

// f(i, a) for every live row i of this thread with its entry a of column e of
// the current tableau; the negated column becomes slot p of np (0 in dropped
// rows).  No barrier.
template <typename T, int NT, typename F>
__device__ __forceinline__ void column(LP<T, NT> &P, int e, F f)
{
    const int m = P.m, N = P.N, p = P.p;
    T *np = P.np;
    const T *pe = P.pr + e;
    // Two rows a turn: their loads from the tableau are in flight together.  (The walk
    // over the window in turns of eight pivots against four: FP32 2,000 LPs of 117 x
    // 150 667 against 705 us, 300 of 16 x 100 90 and 98 us, FP64 within 2 %.)
    for (int i = threadIdx.x; i < m; i += 2 * NT) {
        const int i1 = i + NT;
        const bool two = i1 < m;
        const int ib = two ? i1 : i;
        T a0 = P.tab[int64_t(i) * P.ld + e], a1 = P.tab[int64_t(ib) * P.ld + e];
#pragma unroll 8
        for (int k = 0; k < p; ++k) {
            const T s = pe[k * N];
            a0 = fma(np[k * m + i], s, a0);
            a1 = fma(np[k * m + ib], s, a1);
        }
        const bool l0 = !(P.rowf[i] & ROW_DEAD), l1 = two && !(P.rowf[ib] & ROW_DEAD);
        np[p * m + i] = l0 ? -a0 : T(0);
        if (two) np[p * m + i1] = l1 ? -a1 : T(0);
        if (l0) f(i, a0);
        if (l1) f(i1, a1);
    }
}

// f(j, t) for every column j of this thread with its entry t of row l of the
// current tableau.  No barrier.
template <typename T, int NT, typename F>
__device__ __forceinline__ void row(LP<T, NT> &P, int l, F f)
{
    const int m = P.m, N = P.N, p = P.p;
    const T *pr = P.pr, *nl = P.np + l;
    const T *tl = P.tab + int64_t(l) * P.ld;
    for (int j = threadIdx.x; j < N; j += 2 * NT) {
        const int j1 = j + NT;
        const bool two = j1 < N;
        const int jb = two ? j1 : j;
        T t0 = tl[j], t1 = tl[jb];
#pragma unroll 8
        for (int k = 0; k < p; ++k) {
            const T s = nl[k * m];
            t0 = fma(s, pr[k * N + j], t0);
            t1 = fma(s, pr[k * N + jb], t1);
        }
        f(j, t0);
        if (two) f(j1, t1);
    }
}

// Step 3 for the pivot on (l, e), whose negated column is slot p of np, written
// before a block_pick or a barrier: it becomes slot p of the window, or (P.direct) updates the
// tableau.  de, ne: the entering column's reduced cost and variable.
// f(j, d, b, s) receives every column j of this thread with its new reduced cost
// and variable and, under steepest edge, its weight.  Ends with a barrier only when the workgroup is one wavefront;
// otherwise the next block_pick's or flush's barrier comes before anything
// written here is read by another thread.
template <typename T, int NT, typename F>
__device__ __forceinline__ void push(LP<T, NT> &P, int l, int e, T de, int ne, F f)
{
    const int tid = threadIdx.x;
    const int m = P.m, N = P.N, p = P.p;
    T *np = P.np + p * m, *pr = P.pr + p * N;
    T *tl = P.tab + int64_t(l) * P.ld;
    if constexpr (NT == 64) wave_sync();  // (block_pick has a barrier for larger workgroups)
    const T pe = -np[l];
    const T prhs = P.rhs[l] / pe, pre = T(1) / pe;
    const int bl = uniform(P.basis[l]);
    row(P, l, [&](int j, T t) {
        const T w = j == e ? pre : t / pe;
        const T d = fma(-de, w, j == e ? T(0) : P.obj[j]);
        P.obj[j] = d;
        const int bj = j == e ? bl : P.nonb[j];
        if (!P.steep) f(j, d, bj, T(1));
        tl[j] = w;
        if (!P.direct) {
            pr[j] = w;
            return;
        }
        // The rows of this column, four loads in flight; the squares that steepest
        // edge sums in the order of its own pass (simplex).
        constexpr int R = 16 / int(sizeof(T)), U = 4;
        T *tj = P.tab + j, acc[R];
#pragma unroll
        for (int q = 0; q < R; ++q) acc[q] = T(0);
        for (int i0 = 0; i0 < m; i0 += U) {
            T t[U];
#pragma unroll
            for (int q = 0; q < U; ++q) t[q] = tj[int64_t(min(i0 + q, m - 1)) * P.ld];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const int i = i0 + q;
                if (i >= m) continue;
                if (i != l) {
                    t[q] = fma(np[i], w, j == e ? T(0) : t[q]);
                    tj[int64_t(i) * P.ld] = t[q];
                }
                if (P.steep && !(P.rowf[i] & ROW_DEAD)) acc[q % R] = fma(t[q], t[q], acc[q % R]);
            }
        }
        if (!P.steep) return;
        T s = T(1);
#pragma unroll
        for (int q = 0; q < R; ++q) s += acc[q];
        f(j, d, bj, s);
    });
    P.z = fma(-de, prhs, P.z);
    __syncthreads();  // row l and column e of the window have been read
    for (int i = tid; i < m; i += NT) {
        if (i == l) {
            P.rhs[i] = prhs;
            P.basis[i] = ne;
        } else {
            const T na = np[i];
            P.rhs[i] = fma(na, prhs, P.rhs[i]);
            if (!P.direct) P.tab[int64_t(i) * P.ld + e] = fma(na, pre, T(0));
        }
    }
    if (!P.direct) {
        for (int k = tid; k <= p; k += NT) {
            P.np[k * m + l] = T(0);
            P.pr[k * N + e] = T(0);
        }
        ++P.p;
    }
    if (tid == e % NT) P.nonb[e] = bl;
    if constexpr (NT == 64) __syncthreads();
}

// The sweep: tab takes the window's pivots.  Wavefront w takes row tiles w,
// w + W, ... of sixteen rows, CT column tiles of sixteen a step, the next
// step's loads in flight during this one's products and stores (a tableau in
// device memory is bound by the bytes in flight): one 16 x 16 x 4 matrix
// product per tile and four pivots, whose accumulation is the chain of fmas in
// pivot order.  Operand A holds row 16 rt + lane % 16 and operand B column
// 16 ct + lane % 16 of pivot 4 g + lane / 16.  Rows past m - 1 and columns past
// N - 1 of the last tiles read the last row or column and are not written.
// Starts and ends with a barrier.
template <typename T, int NT>
__device__ __forceinline__ void flush(LP<T, NT> &P)
{
    constexpr int W = NT / 64, CT = 4, GMAX = kMaxWindow / 4;
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6), q = lane >> 4, c16 = lane & 15;
    const int m = P.m, N = P.N, ld = P.ld, p = P.p, G = (p + 3) >> 2;
    __syncthreads();
    if (p == 0) return;
    using Row = typename Tile<T>::V[CT];
    auto place = [&](int rt, int v) { return P.tab + int64_t(min(16 * rt + mfma_row<T>(q, v), m - 1)) * ld; };
    auto load = [&](int rt, int j0, Row &c) {
        static_for<0, 4>([&](auto v) {
            const T *at = place(rt, v);
            static_for<0, CT>([&](auto t) {
                if (j0 + 16 * t < N) c[t][int(v)] = at[min(j0 + 16 * t + c16, N - 1)];
            });
        });
    };
    int rt = wave, j0 = 0;
    Row c;
    T a[GMAX];
    if (16 * rt < m) load(rt, j0, c);
    while (16 * rt < m) {
        int nrt = rt, nj0 = j0 + 16 * CT;
        if (nj0 >= N) { nj0 = 0; nrt += W; }
        Row cn;
        if (16 * nrt < m) load(nrt, nj0, cn);
        if (j0 == 0) {
            const int ia = min(16 * rt + c16, m - 1);
            static_for<0, GMAX>([&](auto g) {
                const int k = 4 * g + q;
                a[g] = T(0);
                if (g < G) {
                    const T x = P.np[min(k, p - 1) * m + ia];
                    a[g] = k < p ? x : T(0);
                }
            });
        }
        static_for<0, GMAX>([&](auto g) {
            if (g >= G) return;
            const T *pk = P.pr + min(4 * g + q, p - 1) * N;
            static_for<0, CT>([&](auto t) {
                if (j0 + 16 * t < N) c[t] = Tile<T>::mma(a[g], pk[min(j0 + 16 * t + c16, N - 1)], c[t]);
            });
        });
        static_for<0, 4>([&](auto v) {
            const int i = 16 * rt + mfma_row<T>(q, v);
            T *at = place(rt, v);
            if (i < m)
                static_for<0, CT>([&](auto t) {
                    const int j = j0 + 16 * t + c16;
                    if (j < N) at[j] = c[t][int(v)];
                });
        });
        static_for<0, CT>([&](auto t) { c[t] = cn[t]; });
        rt = nrt;
        j0 = nj0;
    }
    P.p = 0;
    __syncthreads();
}

// Steps 1-3 until a halt condition.  Returns ST_OPTIMAL, ST_UNBOUNDED or ST_ITER;
// *enter receives the entering Bland index when unbounded.
template <typename T, int NT>
__device__ __forceinline__ int simplex(LP<T, NT> &P, T eps_opt, const SolveParams &prm, int *enter)
{
    const int tid = threadIdx.x;
    const int N = P.N, nm = P.n + P.m;
    const T tol_piv = T(prm.tol_piv);
    int deg_run = 0;
    // Step 1's candidates are collected from the reduced costs, and under steepest
    // edge the weights, as each pivot writes them; the first ones here.
    Best<true, T> in;
    bool bland = prm.k_deg > 0 && deg_run >= prm.k_deg;
    auto offer = [&](int j, T d, int bj, T w) {
        const bool ok = d > eps_opt && bj < nm;
        if (P.steep) {
            const T key = bland ? T(0) : d * d / w;
            in.offer(ok && key == key, key, bj, j);
        } else {
            in.offer(ok, bland ? T(0) : d, bj, j);
        }
    };
    for (int j = tid; j < N; j += NT) {
        T w = T(1);
        if (P.steep) {
            // Steepest edge: d_j^2 / (1 + sum of column j's squares
            // over the live rows); threads walk down their columns,
            // rows i summed into partial sum i mod R, the partial sums
            // then added in order -- the wavefront kernel's order, so
            // both kernels choose the same column.
            constexpr int R = 16 / int(sizeof(T));
            T acc[R];
#pragma unroll
            for (int q = 0; q < R; ++q) acc[q] = T(0);
            for (int i0 = 0; i0 < P.m; i0 += R) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int i = i0 + q;
                    if (i < P.m && !(P.rowf[i] & ROW_DEAD)) {
                        const T t = P.tab[int64_t(i) * P.ld + j];
                        acc[q] = fma(t, t, acc[q]);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < R; ++q) w += acc[q];
        }
        offer(j, P.obj[j], P.nonb[j], w);
    }
    for (;;) {
        if (P.iters >= P.cap) return ST_ITER;
        // Step 1: entering column.
        T key = T(0);
        const int e = block_pick(P, in, key);
        if (e < 0) return ST_OPTIMAL;
        const T de = P.obj[e];
        const int ne = uniform(P.nonb[e]);
        // Step 2: leaving row.
        Best<false, T> out;
        column(P, e, [&](int i, T a) {
            if (a > tol_piv) {
                const T bi = P.rhs[i];
                const T th = (bi > T(0) ? bi : T(0)) / a;
                out.offer(th == th, th, P.basis[i], i);
            }
        });
        T th = T(0);
        const int l = block_pick(P, out, th);
        if (l < 0) { *enter = ne; return ST_UNBOUNDED; }
        if (th == T(0)) { ++deg_run; ++P.degp; } else deg_run = 0;
        bland = prm.k_deg > 0 && deg_run >= prm.k_deg;
        in = Best<true, T>();
        push(P, l, e, de, ne, offer);
        ++P.iters;
        if (P.p == P.K) flush(P);
    }
}

// Whether some reduced cost or right-hand side is not finite, that is, whether the
// window may have held an infinity or NaN: an entry of a pivot's scaled row that
// is not finite makes its column's reduced cost so, for good, and one of its
// column its row's right-hand side.  The caller then solves the LP again with
// every pivot in the tableau at once (P.direct).
template <typename T, int NT>
__device__ __forceinline__ bool overflowed(LP<T, NT> &P)
{
    bool odd = false;
    for (int j = threadIdx.x; j < P.N; j += NT) odd |= !isfinite(P.obj[j]);
    for (int i = threadIdx.x; i < P.m; i += NT) odd |= !isfinite(P.rhs[i]);
    if constexpr (NT == 64) return ballot(odd) != 0;
    if (odd) P.sh->inf = 1;
    __syncthreads();
    return uniform(P.sh->inf) != 0;
}

// A1/A2: non-basic and basic index arrays, then the tableau rows and right-hand
// sides (sign-normalised so every rhs is >= 0, with a -1 surplus entry per >=
// row).  Returns whether this thread saw a non-finite entry of A.
template <typename T, int NT>
__device__ __forceinline__ bool fill_tableau(LP<T, NT> &P)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    constexpr int W = NT / 64;
    const int m = P.m, n = P.n, N = P.N, ld = P.ld;
    T *tab = P.tab;
    P.p = 0;
    for (int j = tid; j < N; j += NT) P.nonb[j] = (j < n) ? j : n + P.colrow[j - n];
    for (int i = tid; i < m; i += NT) {
        P.basis[i] = (row_sense(P.rowf[i]) == LE) ? n + i : n + m + i;
        const double bi = P.b[P.row_of(i)];
        P.rhs[i] = T((P.rowf[i] & ROW_NEG) ? -bi : bi);
    }
    bool bad = false;
    if (!P.rows) {
        // A in flat order, eight loads a thread in flight; stepping by NT
        // elements advances the row by NT / n and the column by NT % n.
        constexpr int U = 8;
        const int mn = m * n, dq = NT / n, dr = NT - dq * n;
        int i = tid / n, j = tid - i * n;
        for (int f0 = tid; f0 < mn; f0 += U * NT) {
            double v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = f0 + u * NT < mn ? P.A[f0 + u * NT] : 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (f0 + u * NT < mn) {
                    bad |= !isfinite(v[u]);
                    tab[int64_t(i) * ld + j] = T((P.rowf[i] & ROW_NEG) ? -v[u] : v[u]);
                }
                i += dq;
                j += dr;
                if (j >= n) { j -= n; ++i; }
            }
        }
    }
    for (int i = wave; i < m; i += W) {
        const double sg = (P.rowf[i] & ROW_NEG) ? -1.0 : 1.0;
        const double *Ai = P.A + (int64_t)P.row_of(i) * n;
        T *row = tab + (int64_t)i * ld;
        if (P.rows)
            for (int j = lane; j < n; j += 64) {
                const double aij = Ai[j];
                bad |= !isfinite(aij);
                row[j] = T(sg * aij);
            }
        for (int j = n + lane; j < N; j += 64) row[j] = (P.colrow[j - n] == i) ? T(-1) : T(0);
    }
    return bad;
}

// Phase II objective row: c priced out over the current basis, rows in order
// (the window must be empty; slot 0 of np holds the basic costs meanwhile).
template <typename T, int NT>
__device__ __forceinline__ void price_out(LP<T, NT> &P)
{
    const int tid = threadIdx.x;
    const int m = P.m, n = P.n, N = P.N, ld = P.ld;
    const T *tab = P.tab;
    T *cbv = P.np;
    bool any = false;
    for (int i = tid; i < m; i += NT) {
        const int bv = P.basis[i];
        const T cb = ((P.rowf[i] & ROW_DEAD) || bv >= n) ? T(0) : T(P.c[bv]);
        cbv[i] = cb;
        any |= cb != T(0);
    }
    // The slack basis, with no cost to price out, skips the walks over the rows
    // (80 x 80: a tenth of a lone LP's time).
    const bool none = block_max<T, NT>(any ? 1.0 : 0.0, P.sh) == 0.0;
    if constexpr (NT == 64) __syncthreads();  // cbv
    const int rows = none ? 0 : m;
    for (int j = tid; j < N; j += NT) {
        const int bj = P.nonb[j];
        T acc = (bj < n) ? T(P.c[bj]) : T(0);
        for (int i = 0; i < rows; ++i) {
            const T cb = cbv[i];
            if (cb != T(0)) acc = fma(-cb, tab[(int64_t)i * ld + j], acc);
        }
        P.obj[j] = acc;
    }
    P.z = T(0);
    for (int i = 0; i < rows; ++i) {
        const T cb = cbv[i];
        if (cb != T(0)) P.z = fma(-cb, P.rhs[i], P.z);
    }
    __syncthreads();
}

// Warm start of an FP64 re-solve from the final basis of the single-precision
// solve of the same LP (basis at warm_basis + P.ro, LP numbering; all rows <=
// after normalisation, so the tableau starts at the slack basis).  Tight rows
// are those whose slack is non-basic in the start basis; every basic
// structural enters, in row order, at the tight row of largest |entry| in its
// column not yet used (ties to the lower row).  Returns false -- the tableau
// then holds some mix and must be rebuilt -- when the start basis is not square
// on its tight rows or a pivot entry falls below tol_piv.  P.colrow (unused
// without surplus columns) holds the tight-row flags; the objective row is
// priced out afterwards.
template <typename T, int NT>
__device__ __forceinline__ bool crash(LP<T, NT> &P, const SolveArgs &a)
{
    const int tid = threadIdx.x;
    const int m = P.m, n = P.n, N = P.N;
    const int32_t *wb = a.warm_basis + P.ro;
    Ctrl<T> *sh = P.sh;
    int *tight = P.colrow;
    for (int i = tid; i < m; i += NT) tight[i] = 1;
    for (int j = tid; j < N; j += NT) P.obj[j] = T(0);
    if (tid == 0) { sh->bad = 0; sh->cnt = 0; }
    __syncthreads();
    int cnt = 0;  // basic structurals minus tight rows, this thread's share
    for (int r = tid; r < m; r += NT) {
        const int v = wb[r];
        if (v < 0 || v >= n + m) sh->bad = 1;  // not a basis of this all-<= LP
        else if (v >= n) tight[v - n] = 0;     // basic slack: its row is not tight
        else ++cnt;
    }
    __syncthreads();
    for (int i = tid; i < m; i += NT) cnt -= tight[i];
    if (cnt) atomicAdd(&sh->cnt, cnt);
    __syncthreads();
    if (uniform(sh->bad) || uniform(sh->cnt) != 0) return false;
    const T tol_piv = T(a.prm.tol_piv);
    for (int r = 0;; ++r) {
        const int v = r < m ? uniform(wb[r]) : 0;
        if (r == m || P.p == P.K) flush(P);
        if (r == m) return true;
        if (v >= n) continue;
        // The structural's column (it must still be non-basic).
        T best = T(0);
        Best<false, T> at;
        for (int j = tid; j < N; j += NT) at.offer(P.nonb[j] == v, T(0), j, j);
        const int c = block_pick(P, at, best);
        if (c < 0) return false;
        // The unused tight row of largest |entry| (ties to the lower row).
        Best<true, T> big;
        column(P, c, [&](int i, T t) { big.offer(tight[i] && t == t, T(fabs(t)), i, i); });
        const int l = block_pick(P, big, best);
        if (l < 0 || !(best > tol_piv)) return false;
        push(P, l, c, T(0), v, [](int, T, int, T) {});
        if (tid == l % NT) tight[l] = 0;
        ++P.iters;
    }
}

// Repair of the crashed start (objective row priced out): the dual simplex
// method, with d_j taken as min(d_j, 0), restores primal feasibility when the
// start is dual feasible up to the single-precision level tol_dual -- leaving
// row: the most negative right-hand side below -tol_p (ties to the smallest
// basic Bland index); entering column: the smallest min(d_j, 0) / t_lj over
// t_lj < -tol_piv (ties to the smallest Bland index) -- then the primal method
// removes any d_j > eps_opt left.  A primal feasible start that is not dual
// feasible goes straight to the primal method.  Returns kPrimal for the caller
// to go on with the primal method, the status when the repair ends otherwise,
// or -1 when the start is neither.
constexpr int kPrimal = -2;
template <typename T, int NT>
__device__ __forceinline__ int dual_repair(LP<T, NT> &P, T tol_dual, T tol_p, const SolveParams &prm)
{
    const int tid = threadIdx.x;
    const int m = P.m, N = P.N, nm = P.n + P.m;
    const T tol_piv = T(prm.tol_piv);
    Ctrl<T> *sh = P.sh;
    // Dual and primal feasibility of the start.
    double dmax = 0.0, pinf = 0.0;
    for (int j = tid; j < N; j += NT)
        if (P.nonb[j] < nm && P.obj[j] > tol_dual) dmax = 1.0;
    for (int i = tid; i < m; i += NT)
        if (!(P.rowf[i] & ROW_DEAD) && P.rhs[i] < -tol_p) pinf = 1.0;
    const bool dual_bad = block_max<T, NT>(dmax, sh) > 0.0;
    const bool primal_bad = block_max<T, NT>(pinf, sh) > 0.0;
    if (dual_bad) return primal_bad ? -1 : kPrimal;
    for (;;) {
        if (P.iters >= P.cap) return ST_ITER;
        T best = T(0);
        Best<true, T> out;
        for (int i = tid; i < m; i += NT) {
            const T v = P.rhs[i];
            out.offer(!(P.rowf[i] & ROW_DEAD) && v < -tol_p, -v, P.basis[i], i);
        }
        const int l = block_pick(P, out, best);
        if (l < 0 || P.p == P.K) flush(P);
        if (l < 0) return kPrimal;  // primal feasible
        Best<false, T> in;
        row(P, l, [&](int j, T t) {
            const int bj = P.nonb[j];
            if (bj < nm && t < -tol_piv) {
                const T d = P.obj[j];
                const T ratio = (d < T(0) ? d : T(0)) / t + T(0);  // +0 for -0
                in.offer(ratio == ratio, ratio, bj, j);
            }
        });
        const int e = block_pick(P, in, best);
        if (e < 0) return ST_INFEASIBLE;  // row l cannot reach its bound
        const T de = P.obj[e];
        const int ne = uniform(P.nonb[e]);
        column(P, e, [](int, T) {});
        __syncthreads();
        push(P, l, e, de, ne, [](int, T, int, T) {});
        ++P.iters;
    }
}

// Solve LP k with the tableau at P.tab (LDS or HBM).  Row classification
// (rowf, colrow, Ctrl counts) has been done by the caller.
template <typename T, int NT>
__device__ __forceinline__ void solve_lp(LP<T, NT> &P, const SolveArgs &a, int placement)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int m = P.m, n = P.n, N = P.N, ld = P.ld;
    Ctrl<T> *sh = P.sh;
    T *tab = P.tab;

    bool bad = fill_tableau<T, NT>(P);
    double cmax = 0.0;
    for (int j = tid; j < n; j += NT) {
        const double cj = P.c[j];
        bad |= !isfinite(cj);
        cmax = fmax(cmax, fabs(cj));
    }
    if (bad) sh->bad = 1;
    double bmax = 0.0;
    for (int i = tid; i < m; i += NT) bmax = fmax(bmax, fabs(P.b[P.row_of(i)]));
    __syncthreads();
    const double cnorm = block_max<T, NT>(cmax, sh);
    const double bnorm = block_max<T, NT>(bmax, sh);
    int status = ST_OPTIMAL, enter = -1;
    const bool invalid = uniform(sh->bad) != 0;
    P.iters = 0; P.it1 = 0; P.degp = 0;
    P.cap = a.prm.max_iters > 0 ? a.prm.max_iters
                                : 50 * (m + n + (m - uniform(sh->neq)) + P.nart);

    // Warm start of an FP64 re-solve from the single-precision solve's final
    // basis of this LP (not for screened solves, whose repair the wavefront
    // kernel does): only when that solve ended optimal -- its status is still
    // in status[k] -- with few violated rows, and only for all-<= LPs.
    // (FP64 only: single-precision solves start from the slack basis.)
    bool warm = sizeof(T) == 8 && !invalid && a.warm_basis && !a.warm_rows && P.nart == 0 && uniform(a.status[P.k]) == ST_OPTIMAL &&
                !(a.warm_viol && uniform(a.warm_viol[P.k]) > a.warm_max_viol);
    if (invalid) status = ST_INVALID;
    for (bool again = false; !invalid;) {
        if (again) {
            // From the slack basis, the tableau rebuilt.
            warm = again = false;
            __syncthreads();
            for (int i = tid; i < m; i += NT) P.rowf[i] &= ~ROW_DEAD;
            if (tid == 0) sh->inf = 0;
            fill_tableau<T, NT>(P);
            P.iters = P.it1 = P.degp = 0;
            enter = -1;
            status = ST_OPTIMAL;
            __syncthreads();
        }
        // A crash that stops part-way leaves a tableau of no use.
        if (sizeof(T) == 8 && warm && (!crash<T, NT>(P, a) || overflowed(P))) {
            again = true;
            continue;
        }
        // Phase I where some row needs an artificial, then Phase II.
        for (int phase = P.nart > 0 ? 1 : 2; status == ST_OPTIMAL; phase = 2) {
            T eps_opt;
            int r = kPrimal;
            if (phase == 1) {
                // Objective row: the sum of the artificial rows (in row order).
                double dmax = 0.0;
                for (int j = tid; j < N; j += NT) {
                    T acc = T(0);
                    for (int i = 0; i < m; ++i)
                        if (row_sense(P.rowf[i]) != LE) acc += tab[(int64_t)i * ld + j];
                    P.obj[j] = acc;
                    dmax = fmax(dmax, fabs(double(acc)));
                }
                P.z = T(0);
                for (int i = 0; i < m; ++i)
                    if (row_sense(P.rowf[i]) != LE) P.z += P.rhs[i];
                __syncthreads();
                eps_opt = T(a.prm.tol_opt * fmax(1.0, block_max<T, NT>(dmax, sh)));
            } else {
                price_out<T, NT>(P);
                eps_opt = T(a.prm.tol_opt * fmax(1.0, cnorm));
                // Single-precision level for the start's reduced costs.
                if (sizeof(T) == 8 && warm)
                    r = dual_repair<T, NT>(P, T(1e-5 * fmax(1.0, cnorm)), T(a.prm.tol_feas * (1.0 + bnorm)), a.prm);
            }
            if (r == kPrimal) r = simplex<T, NT>(P, eps_opt, a.prm, &enter);
            // -1: a start neither primal nor dual feasible.
            if (r == -1 || (!P.direct && overflowed(P))) {
                P.direct |= r != -1;
                again = true;
                break;
            }
            if (phase == 2) {
                status = r;
                break;
            }
            P.it1 = P.iters;
            enter = -1;
            if (r == ST_ITER) status = ST_ITER;
            else if (r == ST_UNBOUNDED) status = ST_NUMERICAL;
            else if (-double(P.z) < -a.prm.tol_feas * (1.0 + bnorm)) status = ST_INFEASIBLE;
            if (status != ST_OPTIMAL) break;
            // Drive basic artificials out, in row order; drop redundant rows.
            const T tol_piv = T(a.prm.tol_piv);
            for (int i = 0;; ++i) {
                if (i == m || P.p == P.K) flush(P);
                if (i == m) break;
                __syncthreads();
                if (uniform(P.basis[i]) < n + m) continue;
                T best = T(0);
                Best<false, T> at;
                row(P, i, [&](int j, T t) {
                    const int bj = P.nonb[j];
                    at.offer(bj < n + m && fabs(t) > tol_piv, T(0), bj, j);
                });
                const int e = block_pick(P, at, best);
                if (e >= 0) {
                    const T de = P.obj[e];
                    const int ne = uniform(P.nonb[e]);
                    column(P, e, [](int, T) {});
                    __syncthreads();
                    push(P, i, e, de, ne, [](int, T, int, T) {});
                } else if (tid == i % NT) {
                    P.rowf[i] |= ROW_DEAD;
                }
            }
            if (!P.direct && overflowed(P)) {
                P.direct = again = true;
                break;
            }
        }
        if (!again) break;
    }

    // A8: extraction.  x_j = rhs of the row where j is basic, else 0;
    // objective recomputed in FP64 from the input c by wavefront 0 in a fixed order.
    __syncthreads();
    T *xv = P.obj;  // reuse as an n-vector
    for (int j = tid; j < n; j += NT) xv[j] = T(0);
    __syncthreads();
    int nbs = 0;
    if (status == ST_OPTIMAL) {
        for (int i = tid; i < m; i += NT) {
            const int bv = P.basis[i];
            if (bv < n && !(P.rowf[i] & ROW_DEAD)) xv[bv] = P.rhs[i];
        }
    }
    __syncthreads();
    const auto &out = *late_args();
    double *x = out.x + P.co;
    if (status == ST_OPTIMAL) {
        for (int j = tid; j < n; j += NT) x[j] = double(xv[j]);
    } else {
        for (int j = tid; j < n; j += NT) x[j] = __builtin_nan("");
    }
    if (wave == 0) {
        double z = 0.0;
        for (int j = lane; j < n; j += 64) {
            const double xj = double(xv[j]);
            z = fma(P.c[j], xj, z);
            nbs += (xj != 0.0);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            z += __shfl_xor(z, off);
            nbs += __shfl_xor(nbs, off);
        }
        if (lane == 0) {
            double objv = z;
            if (status == ST_UNBOUNDED) objv = __builtin_inf();
            else if (status != ST_OPTIMAL) objv = __builtin_nan("");
            out.obj[P.k] = objv;
            out.status[P.k] = status;
            if (out.enter_out) out.enter_out[P.k] = (status == ST_UNBOUNDED) ? enter : -1;
            if (out.stats) {
                int32_t *st = out.stats + 8 * P.k;
                if (out.refine_stats) {
                    st[3] = warm ? 2 : 1;  // 2: started from the single-precision basis
                    st[4] = P.iters;
                } else {
                    st[0] = P.it1;
                    st[1] = P.iters - P.it1;
                    st[2] = P.degp;
                    st[3] = 0;
                    st[4] = 0;
                    st[5] = 0;
                }
                st[6] = placement;
                st[7] = nbs;
            }
        }
    }
    if (out.basis_out)
        for (int i = tid; i < m; i += NT)
            out.basis_out[P.ro + i] = (P.rowf[i] & ROW_DEAD) ? -1 : P.basis[i];
    __syncthreads();
}

// An LP this launch was not planned for (its index arrays or tableau would
// not fit the launch's LDS or device-memory slot): reported NUMERICAL
// without touching the tableau storage.
template <typename T, int NT>
__device__ __forceinline__ void reject_lp(const LP<T, NT> &P, const SolveArgs &a)
{
    const int tid = threadIdx.x;
    for (int j = tid; j < P.n; j += NT) a.x[P.co + j] = __builtin_nan("");
    if (a.basis_out)
        for (int i = tid; i < P.m; i += NT) a.basis_out[P.ro + i] = -1;
    if (tid == 0) {
        a.obj[P.k] = __builtin_nan("");
        a.status[P.k] = ST_NUMERICAL;
        if (a.enter_out) a.enter_out[P.k] = -1;
        if (a.stats) {
            int32_t *st = a.stats + 8 * P.k;
            if (a.refine_stats) {
                st[3] = 1;
                st[4] = 0;
            } else {
                for (int q = 0; q < 8; ++q) st[q] = 0;
            }
        }
    }
}

// STEEP: steepest-edge pricing, a kernel of its own so that its code costs the
// default rule's no registers (in one kernel 500 x 500 FP64 took 8.2 ms, apart 7.3).
template <typename T, int NT, bool STEEP>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void simplex_kernel(SolveArgs a)
{
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    Ctrl<T> *sh = reinterpret_cast<Ctrl<T> *>(smem);
    const int64_t total = a.num_dev ? int64_t(a.id_base) + *a.num_dev : a.num;
    // (Values every thread reads alike are made scalar: the loop bounds, strides
    // and addresses built from them then cost no vector registers.)
    int64_t item = blockIdx.x;
    while (item < total) {
        if (tid == 0) sh->next = gridDim.x + (a.queue ? atomicAdd(a.queue, 1) : 0);
        const int64_t k = a.ids ? int64_t(uniform(a.ids[item])) : item;
        LP<T, NT> P;
        P.k = k;
        if (a.um > 0) {
            P.m = a.um; P.n = a.un;
            P.A = a.A + k * int64_t(a.um) * a.un;
            P.ro = k * a.um;
            P.co = k * a.un;
        } else {
            P.m = uniform(a.m[k]); P.n = uniform(a.n[k]);
            P.A = a.A + uniform64(a.aoff[k]);
            P.ro = uniform64(a.roff[k]);
            P.co = uniform64(a.coff[k]);
        }
        P.b = a.b + P.ro;
        P.c = a.c + P.co;
        P.rows = nullptr;
        P.m_full = P.m;
        const int8_t *sense = a.sense + P.ro;
        if (a.shared) {
            // One LP's constraints shared by the batch (optionally a row subset of them).
            P.A = a.A;
            P.b = a.b;
            sense = a.sense;
            P.m_full = a.m_full;
            P.rows = a.row_subset ? a.row_subset + k * int64_t(P.m) : nullptr;
        }
        const int m = P.m, n = P.n;
        // The arrays that row classification fills; the rest follow once the
        // number of columns is known.
        LdsLayout L = lds_layout(m, n, sizeof(T), sizeof(Ctrl<T>));
        P.sh = sh;
        P.turn = 0;
        P.basis = reinterpret_cast<int *>(smem + L.basis);
        P.rowf = reinterpret_cast<int *>(smem + L.rowf);
        P.colrow = reinterpret_cast<int *>(smem + L.colrow);
        P.rhs = reinterpret_cast<T *>(smem + L.rhs);
        if (L.window(kLeastWindow) > int64_t(a.lds_bytes)) {
            reject_lp<T, NT>(P, a);
            __syncthreads();
            item = uniform(sh->next);
            __syncthreads();
            continue;
        }

        // A1: sign-normalise and classify rows (sense after flipping rows with b < 0).
        if (tid == 0) sh->bad = sh->inf = 0;
        __syncthreads();
        bool bad = false;
        for (int i = tid; i < m; i += NT) {
            const int q = P.row_of(i);
            const double bi = P.b[q];
            const int s = sense[q];
            bad |= !isfinite(bi) || s < LE || s > EQ;
            if (P.rows) bad |= P.rows[i] < 0 || P.rows[i] >= P.m_full;
            const bool neg = bi < 0.0;
            int sen = (s < LE || s > EQ) ? LE : s;
            if (neg && sen != EQ) sen = (sen == LE) ? GE : LE;
            P.rowf[i] = (neg ? ROW_NEG : 0) | (sen << 1);
        }
        if (bad) sh->bad = 1;
        __syncthreads();
        // Surplus columns of >= rows in row order (wavefront ballots), counts.
        if (wave == 0) {
            int ng = 0, nart = 0, neq = 0;
            for (int i0 = 0; i0 < m; i0 += 64) {
                const int i = i0 + lane;
                const int sen = (i < m) ? row_sense(P.rowf[i]) : LE;
                const uint64_t ge = __ballot(i < m && sen == GE);
                const uint64_t ar = __ballot(i < m && sen != LE);
                const uint64_t eq = __ballot(i < m && sen == EQ);
                if (i < m && sen == GE)
                    P.colrow[ng + __popcll(ge & ((uint64_t(1) << lane) - 1))] = i;
                ng += __popcll(ge);
                nart += __popcll(ar);
                neq += __popcll(eq);
            }
            if (lane == 0) { sh->ng = ng; sh->nart = nart; sh->neq = neq; }
        }
        __syncthreads();
        P.N = n + uniform(sh->ng);
        P.nart = uniform(sh->nart);
        L = lds_layout(m, P.N, sizeof(T), sizeof(Ctrl<T>));
        P.nonb = reinterpret_cast<int *>(smem + L.nonb);
        P.obj = reinterpret_cast<T *>(smem + L.obj);
        P.pr = reinterpret_cast<T *>(smem + L.win);
        // The tableau in LDS when it fits beside the least window; the window
        // takes what is left, in whole groups of four.
        const int64_t lds = a.lds_bytes, vec = int64_t(sizeof(T)) * (m + P.N);
        const int64_t in_lds_bytes = lds_tab_bytes(m, P.N, sizeof(T));
        const bool in_lds = !a.force_hbm && L.window(a.least_window) + in_lds_bytes <= lds;
        P.ld = in_lds ? lds_tab_ld(P.N) : slot_tab_ld(P.N, int(sizeof(T)));
        const int64_t room = (lds - L.win - (in_lds ? in_lds_bytes + 16 : 0)) / vec;
        // (Steepest edge reads every column of every pivot's tableau: no window.)
        P.steep = STEEP;
        P.direct = P.steep || (in_lds && m <= kDirectRows);
        const int most = P.direct ? 1 : in_lds ? kMaxWindowLds : kMaxWindow;
        P.K = int(room >= most ? most : room >= 4 ? room & ~int64_t(3) : room < 1 ? 1 : room);
        P.np = P.pr + int64_t(P.K) * P.N;
        P.p = 0;
        const int64_t slot_need = int64_t(sizeof(T)) * m * P.ld;
        if (L.window(kLeastWindow) > lds || (!in_lds && (!a.scratch || slot_need > a.slot_bytes))) {
            reject_lp<T, NT>(P, a);
        } else if (in_lds) {
            P.tab = reinterpret_cast<T *>(smem + L.window(P.K));
            solve_lp<T, NT>(P, a, 3);
        } else {
            P.tab = reinterpret_cast<T *>(a.scratch + int64_t(blockIdx.x) * a.slot_bytes);
            solve_lp<T, NT>(P, a, 2);
        }
        item = uniform(sh->next);
        __syncthreads();
    }
    drain_memory();
    if (tid == 0) finish_launch(a.queue, a.reset_extra);
}

__global__ void zero_i32_kernel(int32_t *p, int count)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x)
        p[i] = 0;
}

template <typename T, int NT>
hipError_t launch_t(const SolveArgs &a, int grid, hipStream_t s)
{
    if (a.prm.pricing == 1)
        hipLaunchKernelGGL((simplex_kernel<T, NT, true>), dim3(grid), dim3(NT), a.lds_bytes, s, a);
    else
        hipLaunchKernelGGL((simplex_kernel<T, NT, false>), dim3(grid), dim3(NT), a.lds_bytes, s, a);
    return hipGetLastError();
}

template <typename T, int NT>
int occ_t(int lds)
{
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, (const void *)simplex_kernel<T, NT, false>,
                                                     NT, lds) != hipSuccess)
        return 0;
    return blocks;
}

}  // namespace

hipError_t launch_zero_i32(int32_t *p, int count, hipStream_t s)
{
    hipLaunchKernelGGL(zero_i32_kernel, dim3(1), dim3(64), 0, s, p, count);
    return hipGetLastError();
}

hipError_t launch_simplex(bool fp32, int nt, const SolveArgs &a, int grid, hipStream_t s)
{
    switch (nt) {
    case 64: return fp32 ? launch_t<float, 64>(a, grid, s) : launch_t<double, 64>(a, grid, s);
    case 128: return fp32 ? launch_t<float, 128>(a, grid, s) : launch_t<double, 128>(a, grid, s);
    case 256: return fp32 ? launch_t<float, 256>(a, grid, s) : launch_t<double, 256>(a, grid, s);
    case 512: return fp32 ? launch_t<float, 512>(a, grid, s) : launch_t<double, 512>(a, grid, s);
    default: return hipErrorInvalidValue;
    }
}

int64_t simplex_ctrl_bytes(bool fp32) { return fp32 ? sizeof(Ctrl<float>) : sizeof(Ctrl<double>); }

hipError_t simplex_configure(int max_lds)
{
    const void *fns[] = {
        (const void *)simplex_kernel<float, 64, false>, (const void *)simplex_kernel<double, 64, false>,
        (const void *)simplex_kernel<float, 128, false>, (const void *)simplex_kernel<double, 128, false>,
        (const void *)simplex_kernel<float, 256, false>, (const void *)simplex_kernel<double, 256, false>,
        (const void *)simplex_kernel<float, 512, false>, (const void *)simplex_kernel<double, 512, false>,
        (const void *)simplex_kernel<float, 64, true>, (const void *)simplex_kernel<double, 64, true>,
        (const void *)simplex_kernel<float, 128, true>, (const void *)simplex_kernel<double, 128, true>,
        (const void *)simplex_kernel<float, 256, true>, (const void *)simplex_kernel<double, 256, true>,
        (const void *)simplex_kernel<float, 512, true>, (const void *)simplex_kernel<double, 512, true>};
    for (const void *f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int simplex_blocks_per_cu(bool fp32, int nt, int lds)
{
    switch (nt) {
    case 64: return fp32 ? occ_t<float, 64>(lds) : occ_t<double, 64>(lds);
    case 128: return fp32 ? occ_t<float, 128>(lds) : occ_t<double, 128>(lds);
    case 256: return fp32 ? occ_t<float, 256>(lds) : occ_t<double, 256>(lds);
    case 512: return fp32 ? occ_t<float, 512>(lds) : occ_t<double, 512>(lds);
    default: return 0;
    }
}

}  // namespace lpb
