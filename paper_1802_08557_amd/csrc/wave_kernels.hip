// wave_kernels.hip -- one 64-wide wavefront per LP for small tableaux.
//
// For LPs with at most 64 non-basic columns and 64*RB rows the whole solve runs
// in a single wavefront with no workgroup barrier:
//   * lane j owns column j: its non-basic variable nonb (Bland index), its
//     objective-row entry d_j and, during a pivot, its pivot-row entry prow_j;
//   * lane i (+64 r) owns row i: its basic variable, sign/sense flags, its
//     right-hand side b_i and its pivot-column entry pcol_i; the objective
//     row's right-hand side (minus the objective value) is a uniform value;
//   * the constraint rows live in LDS, row-major, so that a pivot's row is one
//     contiguous read and its column one read per lane.
// Step 1 is a wavefront DPP/permlane reduction over the lanes' reduced costs;
// Step 2 reads the entering column and reduces the ratios against the
// row-owned right-hand sides; Step 3 keeps the pivot's column and row vectors
// in registers (see Window) and updates the objective row and the right-hand
// sides there; the tableau is swept once per eight pivots, on the matrix cores.
// What bounds it: the dependent chain of each pivot (reductions, a division
// before and after the ratio test, three LDS round trips) at the occupancy the
// tableaux leave -- two wavefronts per SIMD for 50 x 50 FP64, one for 120 x 40 --
// and, for LPs of few pivots, the read of A from HBM (a 50 x 50 batch cut off
// after one pivot takes 0.45 of the 0.82 ms, 4.6 TB/s).  Measured against one or
// two pivots per sweep of a column-major tableau on the vector units (same work
// queue): 1e5 uniform 50 x 50 FP64 1137 -> 840 us, its FP32 solve 940 -> 710 us, 1e5
// support LPs of 120 x 40 FP64 12.8 -> 8.1 ms, screened FP32 2.13 -> 1.63 ms.  (The
// code that solves LPs again which overflow, see overflowed, takes 3, 1, 2 and 0 %
// of these.)
// The arithmetic of every element (fma(-pcol_i, prow_j, t_ij), prow_j =
// t_lj / PE, Phase I and Phase II objective rows summed in row order) is the
// same as in the workgroup kernel, so both give bitwise-identical results.
//
// An LP whose tableau does not fit (too many surplus columns after sign
// normalisation, or too many rows) is appended to the deferred list, which the
// workgroup kernel drains in a following launch.
#include <math.h>

#include "device_common.h"
#include "internal.h"

namespace lpb {
namespace {

// Row stride (in elements) of the row-major LDS tableau with `cols` columns: any
// number that is not a multiple of four, so that the lanes reading one column
// (one element per row) meet at most two to a bank; lanes reading one row are
// consecutive.
template <typename T>
__host__ __device__ constexpr int row_stride(int cols)
{
    return cols & 3 ? cols : cols + 1;
}

// Uniform value of row i from a per-row register array (row i lives in lane i % 64
// of block i / 64).
template <int RB, typename V>
__device__ __forceinline__ V row_get(const V (&arr)[RB], int i)
{
    if constexpr (RB == 1) {
        return lane_get(arr[0], i & 63);
    } else {
        V out = lane_get(arr[0], i & 63);
#pragma unroll
        for (int r = 1; r < RB; ++r)
            if ((i >> 6) == r) out = lane_get(arr[r], i & 63);
        return out;
    }
}

template <typename T, int RB>
struct WaveLP {
    int m, n, N, C, ld, nart;
    int64_t k, ro, co;
    const double *A, *b, *c;
    T *tab;  // row-major: element (i, j) at tab[i * ld + j], columns 0 .. N-1
    int rowf[RB], basis[RB];
    T pcol[RB];
    T rhs[RB];  // right-hand side of row lane + 64 r
    T z;        // right-hand side of the objective row (uniform)
    int rowat[RB], colat;  // row lane + 64 r of tab, column lane (lanes past the last: the last one's)
    int nonb;   // this lane's column
    T d;        // this lane's objective-row entry
    int iters, it1, degp, cap;
    bool keep;  // the tableau is read again when the current phase ends
    bool alone; // no window
};

// Pivots that the tableau in LDS does not hold yet, oldest first in np / pr:
//     t_ij = fma(np[last]_i, pr[last]_j, ... fma(np[0]_i, pr[0]_j, tab_ij) ...)
// with np the negated pivot columns (row owners' registers) and pr the scaled
// pivot rows (column owners' registers).  A pivot's own row and column, which
// it replaces rather than updates, are written to tab at once, and the
// window's entries of that row and column become 0, so every entry goes
// through the same operations in the same order as with one sweep of the
// tableau per pivot.  (Past the range of T the two differ: 0 times infinity leaves
// NaN in an entry that its pivot replaced.  See overflowed.)
//
// Why a window: a pivot reads one column and one row of the tableau, and with
// the window both cost a short chain of fmas on registers.  The sweep, which
// touches every entry, comes once per window -- for a 50 x 50 LP of 9
// pivots hardly at all -- and is then a low-rank update on the matrix cores,
// whose FP64 and FP32 products accumulate as a chain of fmas in k order, bit
// for bit what the separate sweeps would do.
//
// The window holds NG whole groups of four pivots and the group being filled.
template <typename T, int RB>
struct Group {
    T np[4][RB];
    T pr[4];
};
template <typename T, int RB, int NG>
struct Window {
    Group<T, RB> grp[NG + 1];  // the whole groups, oldest first, end at grp[NG - 1]; grp[NG] is being filled
    int n;                     // whole groups
};

// Exchanges rows of sixteen lanes among four registers: on return x[r] holds,
// in lanes 16 k .. 16 k + 15, what lanes 16 r .. 16 r + 15 of x[k] held.
__device__ __forceinline__ void transpose_rows(int &x0, int &x1, int &x2, int &x3)
{
    auto a = __builtin_amdgcn_permlane32_swap(x0, x2, false, false);
    auto b = __builtin_amdgcn_permlane32_swap(x1, x3, false, false);
    auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    x0 = int(c[0]); x1 = int(c[1]); x2 = int(d[0]); x3 = int(d[1]);
}
__device__ __forceinline__ void transpose_rows(float &x0, float &x1, float &x2, float &x3)
{
    int a = __float_as_int(x0), b = __float_as_int(x1), c = __float_as_int(x2), d = __float_as_int(x3);
    transpose_rows(a, b, c, d);
    x0 = __int_as_float(a); x1 = __int_as_float(b); x2 = __int_as_float(c); x3 = __int_as_float(d);
}
__device__ __forceinline__ void transpose_rows(double &x0, double &x1, double &x2, double &x3)
{
    int al = __double2loint(x0), bl = __double2loint(x1), cl = __double2loint(x2), dl = __double2loint(x3);
    int ah = __double2hiint(x0), bh = __double2hiint(x1), ch = __double2hiint(x2), dh = __double2hiint(x3);
    transpose_rows(al, bl, cl, dl);
    transpose_rows(ah, bh, ch, dh);
    x0 = __hiloint2double(ah, al); x1 = __hiloint2double(bh, bl);
    x2 = __hiloint2double(ch, cl); x3 = __hiloint2double(dh, dl);
}

// The sweep of a tableau of NCT column tiles (see flush).
template <int NCT, typename T, int RB, int NG>
__device__ __forceinline__ void flush_tiles(WaveLP<T, RB> &L, const Window<T, RB, NG> &Q, int count)
{
    const int m = L.m, ld = L.ld;
    // (Opaque to the compiler, which otherwise keeps every tile's bounds in
    // scalar registers across the pivots.)
    int q = threadIdx.x >> 4, c16 = threadIdx.x & 15;
    asm volatile("" : "+v"(q), "+v"(c16));
    const bool in = 16 * (NCT - 1) + c16 < L.N;  // this lane's column of the last column tile exists
    const int whole = m >> 4, tail = m & 15;
    // This lane's elements of row tile rt: component v at at[v][16 * column tile].
    // Rows past m - 1 read row m - 1 and are not written.
    struct Ptr { T *p[4]; };
    auto place = [&](int rt) {
        Ptr at;
        static_for<0, 4>([&](auto v) { at.p[v] = L.tab + min(16 * rt + mfma_row<T>(q, v), m - 1) * ld + c16; });
        return at;
    };
    using Row = typename Tile<T>::V[NCT];
    auto load = [&](const Ptr &at, Row &c) {
        static_for<0, NCT>([&](auto ct) {
            if (ct < NCT - 1 || in)
                static_for<0, 4>([&](auto v) { c[ct][int(v)] = at.p[v][16 * ct]; });
        });
    };
    // Operand A of a group from a(group).
    auto update = [&](auto a, Row &c) {
        static_for<0, NG + 1>([&](auto g) {
            if (NG - g >= count) return;
            const T ag = a(Q.grp[g]);
            static_for<0, NCT>([&](auto ct) { c[ct] = Tile<T>::mma(ag, Q.grp[g].pr[ct], c[ct]); });
        });
    };
    Ptr at = place(0);
    Row c;
    static_for<0, NCT>([&](auto ct) { c[ct] = {T(0), T(0), T(0), T(0)}; });
    wave_sync();
    load(at, c);
    // Whole row tiles, the next one's reads in flight during the products.
    static_for<0, 4 * RB>([&](auto rt) {
        if (rt >= whole) return;
        const Ptr next = place(rt + 1);
        Row cn;
        static_for<0, NCT>([&](auto ct) { cn[ct] = {T(0), T(0), T(0), T(0)}; });
        load(next, cn);
        update([&](const Group<T, RB> &g) { return g.np[rt & 3][rt >> 2]; }, c);
        static_for<0, NCT>([&](auto ct) {
            if (ct < NCT - 1 || in)
                static_for<0, 4>([&](auto v) { at.p[v][16 * ct] = c[ct][int(v)]; });
        });
        at = next;
        static_for<0, NCT>([&](auto ct) { c[ct] = cn[ct]; });
    });
    if (tail) {
        update([&](const Group<T, RB> &g) {
            T x = g.np[0][0];
            static_for<1, 4 * RB>([&](auto rt) {
                const T y = g.np[rt & 3][rt >> 2];
                x = rt == whole ? y : x;
            });
            return x;
        }, c);
        static_for<0, NCT>([&](auto ct) {
            if (ct < NCT - 1 || in)
                static_for<0, 4>([&](auto v) {
                    if (mfma_row<T>(q, v) < tail) at.p[v][16 * ct] = c[ct][int(v)];
                });
        });
    }
}

// The sweep: tab takes the window's pivots, the last `count` of its NG + 1
// groups (slots past the last pivot hold 0).  16 x 16 tiles, one rank-4
// matrix product per group: operand A holds row 16 rt + lane % 16 and operand
// B column 16 ct + lane % 16 of the group's pivot lane / 16, which is what its
// registers hold after exchanging their rows of sixteen lanes.  The window's
// registers are used up.
template <typename T, int RB, int NG>
__device__ __forceinline__ void flush(WaveLP<T, RB> &L, Window<T, RB, NG> &Q, int count)
{
    static_for<0, NG + 1>([&](auto g) {
        if (NG - g >= count) return;
        static_for<0, RB>([&](auto r) {
            transpose_rows(Q.grp[g].np[0][r], Q.grp[g].np[1][r], Q.grp[g].np[2][r], Q.grp[g].np[3][r]);
        });
        transpose_rows(Q.grp[g].pr[0], Q.grp[g].pr[1], Q.grp[g].pr[2], Q.grp[g].pr[3]);
    });
    const int nct = (L.N + 15) >> 4;
    if (nct == 4) flush_tiles<4>(L, Q, count);
    else if (nct == 3) flush_tiles<3>(L, Q, count);
    else if (nct == 2) flush_tiles<2>(L, Q, count);
    else flush_tiles<1>(L, Q, count);
    wave_sync();
}

// This lane's rows of column e of the current tableau, S pivots in the group
// being filled (anything past row m - 1).
template <int S, typename T, int RB, int NG>
__device__ __forceinline__ void column(const WaveLP<T, RB> &L, const Window<T, RB, NG> &Q, int e, T (&a)[RB])
{
    static_for<0, RB>([&](auto r) {
        a[r] = L.tab[L.rowat[r] + e];
    });
    static_for<0, NG + 1>([&](auto g) {
        if (g < NG && NG - g > Q.n) return;
        static_for<0, (g < NG ? 4 : S)>([&](auto k) {
            const T s = lane_get(Q.grp[g].pr[k], e);
            static_for<0, RB>([&](auto r) { a[r] = fma(Q.grp[g].np[k][r], s, a[r]); });
        });
    });
}

// This lane's column of row l of the current tableau, S pivots in the group
// being filled (anything past column C - 1).
template <int S, typename T, int RB, int NG>
__device__ __forceinline__ T row(const WaveLP<T, RB> &L, const Window<T, RB, NG> &Q, int l)
{
    T v = L.tab[l * L.ld + L.colat];
    // The block of rows that holds row l, chosen once for all pivots.
    static_for<0, RB>([&](auto r) {
        if (RB > 1 && (l >> 6) != r) return;
        static_for<0, NG + 1>([&](auto g) {
            if (g < NG && NG - g > Q.n) return;
            static_for<0, (g < NG ? 4 : S)>([&](auto k) {
                v = fma(lane_get(Q.grp[g].np[k][r], l & 63), Q.grp[g].pr[k], v);
            });
        });
    });
    return v;
}

// The pivot row of (l, e) scaled: lane j's entry of the new row l, 1 / PE in
// column e.  rowv is its entry of row l, L.pcol holds the pivot column.
template <typename T, int RB>
__device__ __forceinline__ T scaled_row(const WaveLP<T, RB> &L, int l, int e, T rowv)
{
    return (int(threadIdx.x) == e ? T(1) : rowv) / row_get<RB>(L.pcol, l);
}

// Step 3 for the pivot on (l, e) outside the tableau: the objective row, every
// right-hand side and the index arrays are updated in their owners' registers.
// L.pcol holds the pivot column (0 for dead and padding rows), prow the scaled
// row, prow_rhs the scaled right-hand side of row l.
template <typename T, int RB>
__device__ __forceinline__ void advance(WaveLP<T, RB> &L, int l, int e, T prow, T prow_rhs)
{
    const int lane = threadIdx.x;
    const bool at_e = lane == e;
    const T de = lane_get(L.d, e);
    L.d = fma(-de, prow, at_e ? T(0) : L.d);
    L.z = fma(-de, prow_rhs, L.z);
#pragma unroll
    for (int r = 0; r < RB; ++r)
        L.rhs[r] = lane + 64 * r == l ? prow_rhs : fma(-L.pcol[r], prow_rhs, L.rhs[r]);  // (padding rows: 0 stays 0)
}

// The variables of row l and column e change places.
template <typename T, int RB>
__device__ __forceinline__ void swap_index(WaveLP<T, RB> &L, int l, int e)
{
    const int bl = row_get<RB>(L.basis, l);
    const int ne = lane_get(L.nonb, e);
#pragma unroll
    for (int r = 0; r < RB; ++r)
        if (int(threadIdx.x) + 64 * r == l) L.basis[r] = ne;
    if (int(threadIdx.x) == e) L.nonb = bl;
}

// The pivot becomes slot S of the group being filled.  S = 4: the slot is `slot`,
// known at run time, and unused slots hold 0.
template <int S, typename T, int RB, int NG>
__device__ __forceinline__ void push(WaveLP<T, RB> &L, Window<T, RB, NG> &Q, int l, int e, T prow, T prow_rhs,
                                     int slot = S)
{
    const int lane = threadIdx.x;
    const int m = L.m, C = L.C;
    const bool at_e = lane == e;
    advance(L, l, e, prow, prow_rhs);
    const T pre = lane_get(prow, e);
    T *tab = L.tab;
    bool at_l[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const int i = lane + 64 * r;
        at_l[r] = i == l;
        if (i < m) tab[i * L.ld + e] = at_l[r] ? pre : fma(-L.pcol[r], pre, T(0));
    }
    if (lane < C && !at_e) tab[l * L.ld + lane] = prow;
    wave_sync();
    // Row l and column e now come from tab alone.
    static_for<0, NG + 1>([&](auto g) {
        if (g < NG && NG - g > Q.n) return;
        static_for<0, (g < NG ? 4 : S)>([&](auto k) {
            Q.grp[g].pr[k] = at_e ? T(0) : Q.grp[g].pr[k];
            static_for<0, RB>([&](auto r) { Q.grp[g].np[k][r] = at_l[r] ? T(0) : Q.grp[g].np[k][r]; });
        });
    });
    static_for<(S < 4 ? S : 0), (S < 4 ? S + 1 : 4)>([&](auto k) {
        const bool mine = S < 4 || k == slot;
        const T y = at_e ? T(0) : prow, y0 = Q.grp[NG].pr[k];
        Q.grp[NG].pr[k] = mine ? y : y0;
        static_for<0, RB>([&](auto r) {
            const T w = at_l[r] ? T(0) : -L.pcol[r], w0 = Q.grp[NG].np[k][r];
            Q.grp[NG].np[k][r] = mine ? w : w0;
        });
    });
    swap_index(L, l, e);
}

// The pivot in the tableau itself (no pivot waits in a window): row l and column e
// are replaced, every other entry takes its fma.
template <typename T, int RB>
__device__ __forceinline__ void replace(WaveLP<T, RB> &L, int l, int e, T prow, T prow_rhs)
{
    const int lane = threadIdx.x;
    advance(L, l, e, prow, prow_rhs);
    swap_index(L, l, e);
    static_for<0, RB>([&](auto r) {
        const int rows = min(L.m - 64 * r, 64);
#pragma unroll 2
        for (int i = 0; i < rows; ++i) {
            const T a = lane_get(L.pcol[r], i);
            T *at = L.tab + (64 * r + i) * L.ld + L.colat;
            const T t = *at, v = 64 * r + i == l ? prow : fma(-a, prow, lane == e ? T(0) : t);
            if (lane < L.C) *at = v;
        }
    });
    wave_sync();
}

// The same for steepest edge, which reads every column of every pivot's tableau:
// returns this lane's weight in the new one (weight), so that no pass of its own is
// left to Step 1.  Every lane stays active, those past the last column repeating it
// to the store, because the row owners' entries are read across lanes.
template <typename T, int RB>
__device__ __forceinline__ T replace_and_weigh(WaveLP<T, RB> &L, int l, int e, T prow, T prow_rhs)
{
    const int lane = threadIdx.x;
    advance(L, l, e, prow, prow_rhs);
    swap_index(L, l, e);
    prow = L.colat == e ? lane_get(prow, e) : prow;
    // Column e starts from 0, and row l from its new entries with a multiplier of 0
    // (0 times infinity is NaN: a scaled row that is not finite has row l left out).
    T np[RB];
    static_for<0, RB>([&](auto r) {
        if (lane + 64 * r < L.m) L.tab[(lane + 64 * r) * L.ld + e] = T(0);
        np[r] = lane + 64 * r == l ? T(0) : -L.pcol[r];
    });
    if (lane < L.C) L.tab[l * L.ld + lane] = prow;
    wave_sync();
    const bool skip_l = ballot(!isfinite(prow)) != 0;
    constexpr int R = 16 / int(sizeof(T)), U = 8;
    T acc[R];
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] = T(0);
    static_for<0, RB>([&](auto r) {
        const int rows = min(L.m - 64 * r, 64);
        const uint64_t dead = ballot((L.rowf[r] & kRowDead) != 0);
        uint64_t odd = dead;  // rows whose group of U takes a look at each
        if (skip_l && (l >> 6) == r) odd |= uint64_t(1) << (l & 63);
        for (int i0 = 0; i0 < rows; i0 += U) {
            T *at = L.tab + (64 * r + i0) * L.ld + L.colat;
            if (i0 + U <= rows && !((odd >> i0) & 0xff)) {
                T t[U];
#pragma unroll
                for (int q = 0; q < U; ++q) t[q] = at[q * L.ld];
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    t[q] = fma(lane_get(np[r], i0 + q), prow, t[q]);
                    acc[q % R] = fma(t[q], t[q], acc[q % R]);
                }
#pragma unroll
                for (int q = 0; q < U; ++q) at[q * L.ld] = t[q];
                continue;
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                if (i0 + q >= rows) continue;
                const T a = lane_get(np[r], i0 + q), t0 = at[q * L.ld];
                const T t = 64 * r + i0 + q == l ? prow : fma(a, prow, t0);
                at[q * L.ld] = t;
                if (!((dead >> (i0 + q)) & 1)) acc[q % R] = fma(t, t, acc[q % R]);
            }
        }
    });
    wave_sync();
    T w = T(1);
#pragma unroll
    for (int q = 0; q < R; ++q) w += acc[q];
    return w;
}

// Whether some reduced cost or right-hand side is not finite, that is, whether the
// window may have held an infinity or NaN: an entry of a pivot's scaled row that
// is not finite makes its column's reduced cost so, for good, and one of its
// column its row's right-hand side.  The caller then solves the LP again with
// every pivot in the tableau at once (L.alone).
template <typename T, int RB>
__device__ __forceinline__ bool overflowed(const WaveLP<T, RB> &L)
{
    bool odd = !isfinite(L.d);
    static_for<0, RB>([&](auto r) { odd |= !isfinite(L.rhs[r]); });
    return ballot(odd) != 0;
}

constexpr int kAgain = 64;  // the status of such an LP until then

// Slots S .. 3 of the group being filled hold no pivot.
template <int S, typename T, int RB>
__device__ __forceinline__ void pad_group(Group<T, RB> &g)
{
    static_for<S, 4>([&](auto k) {
        g.pr[k] = T(0);
        static_for<0, RB>([&](auto r) { g.np[k][r] = T(0); });
    });
}

// The group being filled becomes the window's newest whole group.
template <typename T, int RB, int NG>
__device__ __forceinline__ void keep_group(Window<T, RB, NG> &Q)
{
    static_for<0, NG>([&](auto g) {
        static_for<0, 4>([&](auto k) {
            Q.grp[g].pr[k] = Q.grp[g + 1].pr[k];
            static_for<0, RB>([&](auto r) { Q.grp[g].np[k][r] = Q.grp[g + 1].np[k][r]; });
        });
    });
    ++Q.n;
}

// The pivots of a warm start (crash, dual simplex): a window whose slots are
// filled one at a time, unused ones 0.
template <typename T, int RB, int NG>
struct Pending {
    Window<T, RB, NG> Q;
    int s;  // pivots in Q.grp[NG]
    __device__ __forceinline__ void clear()
    {
        Q.n = 0;
        s = 0;
        pad_group<0>(Q.grp[NG]);
    }
    // Loads column e into the per-row pivot-column registers (0 for dropped rows).
    __device__ __forceinline__ void load_pcol(WaveLP<T, RB> &L, int e)
    {
        T a[RB];
        column<4>(L, Q, e, a);
#pragma unroll
        for (int r = 0; r < RB; ++r) L.pcol[r] = (L.rowf[r] & (kRowDead | kRowPad)) ? T(0) : a[r];
    }
    __device__ __forceinline__ T load_row(WaveLP<T, RB> &L, int l) { return row<4>(L, Q, l); }
    // Pivot on (l, e) whose column is in L.pcol and whose row is rowv.
    __device__ __forceinline__ void pivot(WaveLP<T, RB> &L, int l, int e, T rowv)
    {
        push<4>(L, Q, l, e, scaled_row(L, l, e, rowv), row_get<RB>(L.rhs, l) / row_get<RB>(L.pcol, l), s);
        if (++s < 4 || Q.n == NG) return;
        keep_group(Q);
        s = 0;
        pad_group<0>(Q.grp[NG]);
    }
    __device__ __forceinline__ bool full() const { return s == 4; }
    // Brings the tableau in LDS up to date.
    __device__ __forceinline__ void sweep(WaveLP<T, RB> &L)
    {
        flush(L, Q, Q.n + 1);
        clear();
    }
};

// Step 1: the entering column (wavefront-uniform), or -1 when none is eligible.
// Dantzig: the largest d_j (positive where eligible, so its bits order like
// an unsigned integer's), ties to the smallest Bland index; Bland: the smallest
// eligible Bland index.
template <typename T>
__device__ __forceinline__ int price(bool elig, T d, int nonb, bool bland)
{
    const uint64_t any = ballot(elig);
    if (!any) return -1;
    uint64_t tied = any;
    if (!bland) {
        tied = wave_max_nonneg(elig, d);
        if (__builtin_expect(__popcll(tied) == 1, 1)) return __builtin_ctzll(tied);
    }
    const bool in = (tied >> (threadIdx.x & 63)) & 1;
    const int bmin = wave_min_i(in ? nonb : kBig);
    return __builtin_ctzll(ballot(in && nonb == bmin));
}

// Weight of steepest edge: 1 + the sum of the squares of this lane's column over the
// live rows, row i into partial sum i mod R (the workgroup kernel's order).
template <typename T, int RB>
__device__ __forceinline__ T weight(const WaveLP<T, RB> &P)
{
    constexpr int R = 16 / int(sizeof(T)), U = 8;
    T acc[R];
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] = T(0);
    static_for<0, RB>([&](auto r) {
        const int rows = min(P.m - 64 * r, 64);
        const uint64_t dead = ballot((P.rowf[r] & kRowDead) != 0);
#pragma unroll 1
        for (int i0 = 0; i0 < rows; i0 += U) {
            const T *at = P.tab + (64 * r + i0) * P.ld + P.colat;
            T t[U];
#pragma unroll
            for (int q = 0; q < U; ++q) t[q] = at[min(q, rows - 1 - i0) * P.ld];
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (i0 + q < rows && !((dead >> (i0 + q)) & 1)) acc[q % R] = fma(t[q], t[q], acc[q % R]);
        }
    });
    T w = T(1);
#pragma unroll
    for (int q = 0; q < R; ++q) w += acc[q];
    return w;
}

// Step 1 by steepest edge from this lane's weight.  (A key that is not a number --
// both its terms overflowed -- is not eligible.)
template <typename T, int RB>
__device__ __forceinline__ int price_steepest(const WaveLP<T, RB> &P, bool elig, T w)
{
    const T key = P.d * P.d / w;
    elig &= key == key;
    if (!ballot(elig)) return -1;
    const T best = wave_max_f(elig ? key : -t_inf<T>());
    const uint64_t tied = ballot(elig && key == best);
    if (__popcll(tied) == 1) return __builtin_ctzll(tied);
    const bool in = (tied >> threadIdx.x) & 1;
    const int bmin = wave_min_i(in ? P.nonb : kBig);
    return __builtin_ctzll(ballot(in && P.nonb == bmin));
}

// One iteration with S pivots in the group being filled.  Returns -1 to go
// on, else the status (the group then still holds S pivots).  ALONE: the pivot
// goes to the tableau itself.  STEEP: steepest edge, *w this lane's weight.
template <int S, bool STEEP, bool ALONE = false, typename T, int RB, int NG>
__device__ __forceinline__ int step(WaveLP<T, RB> &P, Window<T, RB, NG> &Q, T eps_opt, const SolveParams &prm,
                                    int &deg_run, int *enter, T *w = nullptr)
{
    const int lane = threadIdx.x;
    if (P.iters >= P.cap) return kIterLimit;
    const bool bland = prm.k_deg > 0 && deg_run >= prm.k_deg;
    // Step 1.
    const bool elig = lane < P.N && P.d > eps_opt && P.nonb < P.n + P.m;
    int e;
    if (STEEP && !bland) e = price_steepest<T, RB>(P, elig, *w);
    else e = price<T>(elig, P.d, P.nonb, bland);
    if (e < 0) return kOptimal;
    // Step 2: each lane's best row (ties to the smaller basic index), then
    // the wavefront minimum ratio, ties to the smallest basic index.
    T a[RB];
    column<S>(P, Q, e, a);
    const T tol_piv = T(prm.tol_piv);
    T th_loc = t_inf<T>();
    int bb_loc = kBig, row_loc = -1;
    bool cand = false;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        const bool live = !(P.rowf[r] & (kRowDead | kRowPad));
        P.pcol[r] = live ? a[r] : T(0);
        // (The division runs on every lane: a branch around it costs more.)
        T th = (P.rhs[r] > T(0) ? P.rhs[r] : T(0)) / a[r];
        asm("" : "+v"(th));
        const int bb = P.basis[r];
        const bool ok = live && a[r] > tol_piv && th == th;
        const bool take = ok && (r == 0 || !cand || th < th_loc || (th == th_loc && bb < bb_loc));
        th_loc = take ? th : th_loc;
        bb_loc = take ? bb : bb_loc;
        row_loc = take ? int(threadIdx.x) + 64 * r : row_loc;
        cand |= ok;
    }
    if (!ballot(cand)) { *enter = lane_get(P.nonb, e); return kUnbounded; }
    const uint64_t tied = wave_min_nonneg(cand, th_loc);
    int src;
    if (__builtin_expect(__popcll(tied) == 1, 1)) {
        src = __builtin_ctzll(tied);
    } else {
        const bool in = (tied >> lane) & 1;
        const int bmin = wave_min_i(in ? bb_loc : kBig);
        src = __builtin_ctzll(ballot(in && bb_loc == bmin));
    }
    const int l = RB == 1 ? src : lane_get(row_loc, src);
    const T th = lane_get(th_loc, src);
    if (th == T(0)) { ++deg_run; ++P.degp; } else deg_run = 0;
    const T prow = scaled_row(P, l, e, row<S>(P, Q, l));
    // The scaled right-hand side of row l is the ratio itself where it is positive.
    const T bl = row_get<RB>(P.rhs, l);
    T prow_rhs = th;
    if (!(bl > T(0))) prow_rhs = bl / row_get<RB>(P.pcol, l);
    if constexpr (STEEP) *w = replace_and_weigh(P, l, e, prow, prow_rhs);
    else if constexpr (ALONE) replace(P, l, e, prow, prow_rhs);
    else push<S>(P, Q, l, e, prow, prow_rhs);
    ++P.iters;
    return -1;
}

// Steps S .. 3 of a group.  Returns -1 to go on with the next group, else the
// status; the group's unused slots then hold 0.
template <int S, typename T, int RB, int NG>
__device__ __forceinline__ int run_group(WaveLP<T, RB> &P, Window<T, RB, NG> &Q, T eps_opt, const SolveParams &prm,
                                         int &deg_run, int *enter)
{
    if constexpr (S < 4) {
        const int r = step<S, false>(P, Q, eps_opt, prm, deg_run, enter);
        if (r >= 0) {
            pad_group<S>(Q.grp[NG]);
            return r;
        }
        return run_group<S + 1>(P, Q, eps_opt, prm, deg_run, enter);
    }
    return -1;
}

template <bool STEEP, typename T, int RB, int NG>
__device__ __forceinline__ int simplex(WaveLP<T, RB> &P, T eps_opt, const SolveParams &prm, int *enter)
{
    int deg_run = 0;
    Window<T, RB, NG> Q;
    Q.n = 0;
    if constexpr (STEEP) {
        T w = weight(P);
        for (;;) {
            const int r = step<0, true, true>(P, Q, eps_opt, prm, deg_run, enter, &w);
            if (r >= 0) return r;
        }
    }
    if (!STEEP && P.alone)
        for (;;) {
            const int r = step<0, false, true>(P, Q, eps_opt, prm, deg_run, enter);
            if (r >= 0) return r;
        }
    for (;;) {
        const int r = run_group<0>(P, Q, eps_opt, prm, deg_run, enter);
        if (r >= 0 && overflowed(P)) return kAgain;
        if (r >= 0 && !P.keep) return r;
        if (r >= 0 || Q.n == NG) {
            flush(P, Q, Q.n + 1);
            Q.n = 0;
            if (r >= 0) return r;
        } else {
            keep_group(Q);
        }
    }
}

// Warm start from a final basis of a single-precision solve: either of a
// relaxation solved on a subset of the rows (warm_rows set: warm_m rows per
// LP, its basis at warm_basis + k * warm_m in relaxation numbering) or of the
// LP itself (warm_rows NULL: its basis at warm_basis + P.ro, LP numbering).
// All rows are <= after normalisation, so the tableau starts at the slack
// basis.  The start basis holds its basic structurals and the slacks of some
// of its rows; the other rows ("tight": slack non-basic) must lose their
// slacks.  Crash: every basic structural enters, in row order, at the tight
// row of largest |entry| in its column not yet used; the full LP's basis then
// is the start basis plus the slacks of any omitted rows.  Returns false when
// a pivot entry falls below tol_piv or the start basis is not square on its
// tight rows.
template <typename T, int RB, int NG>
__device__ __forceinline__ bool crash(WaveLP<T, RB> &P, Pending<T, RB, NG> &W, const SolveArgs &a, int64_t k)
{
    const int lane = threadIdx.x;
    const int n = P.n, m = P.m;
    const int wm = a.warm_rows ? a.warm_m : m;
    const int32_t *wb = a.warm_rows ? a.warm_basis + k * int64_t(wm) : a.warm_basis + P.ro;
    const int32_t *wr = a.warm_rows ? a.warm_rows + k * int64_t(wm) : nullptr;
    const T tol_piv = T(a.prm.tol_piv);
    uint64_t cand[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) cand[r] = 0;
    int nstruct = 0;
    // Tight rows: the start basis's rows, less those whose slack is basic.
    for (int r0 = 0; r0 < wm; r0 += 64) {
        const int r = r0 + lane;
        int q = -1, v = -1, qs = -1;
        if (r < wm) {
            q = wr ? wr[r] : r;
            v = wb[r];
            if (v >= n && v < n + wm) qs = wr ? wr[v - n] : v - n;  // the row of a basic slack
        }
        nstruct += __popcll(ballot(r < wm && v >= 0 && v < n));
        for (int pass = 0; pass < 2; ++pass) {
            const int qq = pass == 0 ? q : qs;
            uint64_t bits = ballot(qq >= 0 && qq < m);
            while (bits) {
                const int src = __builtin_ctzll(bits);
                bits &= bits - 1;
                const int qi = lane_get(qq, src);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    if ((qi >> 6) == rb) {
                        if (pass == 0) cand[rb] |= uint64_t(1) << (qi & 63);
                        else cand[rb] &= ~(uint64_t(1) << (qi & 63));
                    }
            }
        }
    }
    int ntight = 0;
#pragma unroll
    for (int r = 0; r < RB; ++r) ntight += __popcll(cand[r]);
    if (ntight != nstruct) return false;
    int r0 = -64, v = -1;
    uint64_t bits = 0;
    for (;;) {
        // The next basic structural, in row order.
        while (!bits && r0 + 64 < wm) {
            r0 += 64;
            v = r0 + lane < wm ? wb[r0 + lane] : -1;
            bits = ballot(v >= 0 && v < n);
        }
        if (!bits || W.full()) W.sweep(P);
        if (!bits) return true;
        const int src = __builtin_ctzll(bits);
        bits &= bits - 1;
        const int j = lane_get(v, src);
        const uint64_t at = ballot(P.nonb == j);
        if (!at) return false;  // listed twice
        const int c = __builtin_ctzll(at);
        W.load_pcol(P, c);
        T best = T(-1);
        int rl = -1;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int i = lane + 64 * rb;
            if (i < m && ((cand[rb] >> lane) & 1)) {
                const T t = fabs(P.pcol[rb]);
                if (t > best) { best = t; rl = i; }
            }
        }
        const T bmax = wave_max_f(best);
        if (!(bmax > tol_piv)) return false;
        const int l = lane_get(rl, __builtin_ctzll(ballot(rl >= 0 && best == bmax)));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            if ((l >> 6) == rb) cand[rb] &= ~(uint64_t(1) << (l & 63));
        W.pivot(P, l, c, W.load_row(P, l));
        ++P.iters;
    }
}

// Repair of a start basis from a single-precision solve (the final basis of
// an FP32 relaxation, or of the FP32 solve of the LP itself), which the FP64
// arithmetic may find slightly primal or dual infeasible.  A start that is
// dual feasible up to the single-precision level: the dual simplex method,
// with d_j taken as min(d_j, 0), restores primal feasibility -- the leaving
// row is the most negative right-hand side below -tol_p (ties to the smallest
// basic Bland index), the entering column the smallest min(d_j, 0) / t_lj over
// t_lj < -tol_piv (ties to the smallest Bland index) -- and the primal method
// then removes any d_j > eps_opt left.  A start that is primal feasible but
// not dual feasible goes straight to the primal method.  Returns kPrimal for
// the caller to go on with the primal method, the status when the repair ends
// otherwise, or -1 when the start is neither (the caller then solves from the
// slack basis).
constexpr int kPrimal = -2;
template <typename T, int RB, int NG>
__device__ __forceinline__ int dual_repair(WaveLP<T, RB> &P, Pending<T, RB, NG> &W, T tol_dual, T tol_p, const SolveParams &prm)
{
    const int lane = threadIdx.x;
    const int m = P.m, N = P.N, nm = P.n + P.m;
    const T tol_piv = T(prm.tol_piv);
    if (ballot(lane < N && P.d > tol_dual && P.nonb < nm)) {
        bool infeas = false;
#pragma unroll
        for (int r = 0; r < RB; ++r)
            infeas |= lane + 64 * r < m && !(P.rowf[r] & (kRowDead | kRowPad)) && P.rhs[r] < -tol_p;
        if (ballot(infeas)) return -1;
        return kPrimal;
    }
    for (;;) {
        if (P.iters >= P.cap) return kIterLimit;
        T vl = t_inf<T>();
        int bl = kBig, rl = -1;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = lane + 64 * r;
            const T v = P.rhs[r];
            if (i < m && !(P.rowf[r] & (kRowDead | kRowPad)) && v < -tol_p &&
                (v < vl || (v == vl && P.basis[r] < bl))) {
                vl = v; bl = P.basis[r]; rl = i;
            }
        }
        const bool feasible = !ballot(rl >= 0);
        if (feasible || W.full()) W.sweep(P);
        if (feasible) return overflowed(P) ? kAgain : kPrimal;
        const T vmin = wave_min_f(vl);
        const uint64_t tied = ballot(rl >= 0 && vl == vmin);
        int src = __builtin_ctzll(tied);
        if (__popcll(tied) > 1) {
            const bool in = (tied >> lane) & 1;
            const int bmin = wave_min_i(in ? bl : kBig);
            src = __builtin_ctzll(ballot(in && bl == bmin));
        }
        const int l = lane_get(rl, src);
        const T tlj = W.load_row(P, l);
        const T ratio = (P.d < T(0) ? P.d : T(0)) / tlj;
        const bool el = lane < N && P.nonb < nm && tlj < -tol_piv && ratio == ratio;
        if (!ballot(el)) return kInfeasible;  // row l cannot reach its bound
        const T rmin = wave_min_f(el ? ratio : t_inf<T>());
        const uint64_t rt = ballot(el && ratio == rmin);
        int e = __builtin_ctzll(rt);
        if (__popcll(rt) > 1) {
            const bool in = (rt >> lane) & 1;
            const int bmin = wave_min_i(in ? P.nonb : kBig);
            e = __builtin_ctzll(ballot(in && P.nonb == bmin));
        }
        W.load_pcol(P, e);
        W.pivot(P, l, e, tlj);
        ++P.iters;
    }
}

// Bytes of LDS the wave kernel keeps in front of the tableau: the surplus
// column -> row map and the row -> constraint map of a screened LP.  (The
// objective c stays in registers and is fetched across lanes with
// ds_bpermute; x is staged in the tableau's first columns once the pivots are
// done.)  Keeping this small lets one more 50 x 50 FP64 LP fit per CU.
__host__ __device__ constexpr int64_t wave_aux_bytes(int rb, bool gather)
{
    return align16(4 * 64 * rb) + (gather ? align16(4 * 64 * rb) : 0);
}

// Doubles of A each lane prefetches: LPs of up to 64 rows with m * n <= 64 * NPF have
// their whole constraint matrix loaded into registers one LP ahead.  Batches of
// larger (or row-gathered) LPs use the instantiation without the prefetch
// registers.  (With two rows a lane the window leaves no registers for it: FP64 spilled
// 72, 20,000 LPs of 100 x 25 434 us with prefetch, 282 without, of 66 x 4 178 and 90;
// FP32, which did not spill, 400 and 391, 206 and 165.)
constexpr int NPF = 40;

// An LP's geometry and input data, loaded into registers ahead of its solve.
template <int RB, int PFD>
struct Fetch {
    int64_t k, ro, co;
    int m, n;
    const double *A;
    bool has_a;
    double av[PFD > 0 ? PFD : 1];  // A in flat row-major order, element lane + 64 t
    double bv[RB];   // b of row lane + 64 r
    int sv[RB];      // sense of row lane + 64 r
    int rid[RB];     // constraint of the shared LP that row lane + 64 r is (shared only)
    bool bad_row;    // a row index outside the shared LP (this lane's rows)
    double cv;       // c of column lane
};

// Issues the loads of work item `item`.  The LP's geometry is wavefront-uniform
// (computed, or read and broadcast for batches of mixed sizes); every data
// load is an unconditional buffer load through a uniform descriptor whose
// range check returns 0 past the LP's end, so no branch separates the loads and
// nothing waits for them before their first use in the next LP's setup.
template <int RB, int PFD>
__device__ __forceinline__ void fetch(int64_t item, Fetch<RB, PFD> &F)
{
    const auto &a = *late_args();
    const int lane = threadIdx.x;
    const int64_t k = a.ids ? int64_t(uniform(a.ids[item])) : item;
    F.k = k;
    int m, n;
    int64_t aoff;
    if (a.um > 0) {
        m = a.um; n = a.un;
        aoff = k * int64_t(m) * n;
        F.ro = k * m;
        F.co = k * n;
    } else {
        // All five loads in flight before the first broadcast waits for them.
        const int mk = a.m[k], nk = a.n[k];
        const int64_t ak = a.aoff[k], rk = a.roff[k], ck = a.coff[k];
        m = uniform(mk); n = uniform(nk);
        aoff = uniform64(ak);
        F.ro = uniform64(rk);
        F.co = uniform64(ck);
    }
    F.m = m; F.n = n;
    F.A = a.shared ? a.A : a.A + aoff;
    F.bad_row = false;
    if (a.shared) {
        // One LP's constraints shared by the batch; a screened LP takes the
        // rows its subset names (gathered, so A is read row by row later).
        const int32_t *sub = a.row_subset ? a.row_subset + k * int64_t(m) : nullptr;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = lane + 64 * r;
            int q = i;
            if (sub && i < m) q = sub[i];
            const bool okq = q >= 0 && q < a.m_full;
            F.bad_row |= i < m && !okq;
            q = okq ? q : 0;
            F.rid[r] = q;
            F.bv[r] = (i < m) ? a.b[q] : 0.0;
            F.sv[r] = (i < m) ? int(a.sense[q]) : 0;
        }
    } else {
        const __amdgpu_buffer_rsrc_t rb = buffer_over(a.b + F.ro, m * int(sizeof(double)));
        const __amdgpu_buffer_rsrc_t rsn = buffer_over(a.sense + F.ro, m);
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = lane + 64 * r;
            F.rid[r] = i;
            F.bv[r] = buffer_f64(rb, i * int(sizeof(double)));
            F.sv[r] = int(int8_t(__builtin_amdgcn_raw_buffer_load_b8(rsn, i, 0, 0)));
        }
    }
    F.cv = buffer_f64(buffer_over(a.c + F.co, n * int(sizeof(double))), lane * int(sizeof(double)));
    const int mn = m * n;
    F.has_a = PFD > 0 && mn <= 64 * PFD && !(a.shared && a.row_subset);
    if constexpr (PFD > 0) if (F.has_a) {
        const __amdgpu_buffer_rsrc_t rs = buffer_over(F.A, mn * int(sizeof(double)));
#pragma unroll
        for (int t = 0; t < PFD; ++t) F.av[t] = buffer_f64(rs, (lane + 64 * t) * int(sizeof(double)));
    }
}

// Whole groups of four pivots that a window holds besides the one being filled:
// eight pivots per sweep.  Twelve and sixteen were slower, the longer chains
// and the registers costing more than the sweeps they save (1e5 support LPs of
// 120 x 40 FP64 7.95 / 8.14 / 8.70 ms; 1e5 screened FP32 1.57 / 1.72 / 1.95 ms;
// 1e5 uniform 50 x 50 FP64 0.83 / 0.83 / 1.00 ms).
constexpr int kGroups = 1;

// Wavefronts per SIMD that the registers are allotted for.  FP64 without prefetch: two
// hold everything in registers, three spill (20,000 LPs of 60 x 60 417 us with three, 396
// with two, of 50 x 64 349 and 334).  The repair kernel spills 190 registers at three and
// none at two, with two blocks of rows 70 at two and none at one, and 65 to 128 rows
// leave LDS for one wavefront per SIMD anyway.  FP32: five
// (one block of rows) and four spill a few registers outside the pivots, which costs less
// than a wavefront (screened 120 x 40 3.95 ms with five, 3.99 with four).
template <typename T, int RB, int PFD, bool WARM>
constexpr int kWavesPerSimd = PFD > 0 ? 2 : WARM ? 3 - RB : sizeof(T) == 8 ? 2 : 6 - RB;

// STEEP: steepest-edge pricing, apart so that its code costs the default rule's no
// registers (in one kernel 100,000 LPs of 50 x 50 FP64 took 9 % longer), nor the
// window those of steepest edge, which has none (20,000 of 20 x 20 157 us with both
// in one, 118 apart).
template <typename T, int RB, int PFD, bool WARM = false, bool STEEP = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWavesPerSimd<T, RB, PFD, WARM>))) void simplex_wave_kernel(SolveArgs a)
{
    extern __shared__ __align__(16) char smem[];
    constexpr int NG = kGroups;
    const int lane = threadIdx.x;
    int *colrow = reinterpret_cast<int *>(smem);
    int *rowid = reinterpret_cast<int *>(smem + align16(4 * 64 * RB));
    const int64_t aux = wave_aux_bytes(RB, a.shared && a.row_subset);
    const int64_t total = a.num_dev ? int64_t(a.id_base) + *a.num_dev : a.num;
    // The next work item is always known one LP ahead, so its data can be in
    // flight while the current LP pivots.
    const QueuePlace queue(blockIdx.x, gridDim.x);
    int64_t cur = blockIdx.x, nxt = queue.second(blockIdx.x);
    Fetch<RB, PFD> F;
    if (cur < total) fetch<RB, PFD>(cur, F);
    // LPs to solve again pivot by pivot (see overflowed): a list through their
    // status entries, taken up when the work items have run out.
    int redo = -1;
    int alone = 0;  // 1: cur is one of them
    while (cur < total) {
        asm volatile("" : "+v"(alone));  // (opaque, or the loop is copied for either value)
        alone = uniform(alone);
        int qv = 0;
        if (lane == 0 && a.queue) qv = queue.pop(a.queue);
        const int64_t k = F.k;
        // The step to the LP that F was loaded with.
        auto next_item = [&] {
            if (nxt < total) {
                cur = nxt;
                nxt = queue.item(lane_get(qv, 0));
            } else if (!STEEP && redo >= 0) {
                const volatile int32_t *link = a.status;
                cur = redo;
                redo = uniform(link[a.ids ? int64_t(uniform(a.ids[cur])) : cur]);
                alone = 1;
            } else {
                cur = total;
            }
        };
        WaveLP<T, RB> P;
        P.k = k;
        P.m = F.m; P.n = F.n;
        P.A = F.A;
        P.ro = F.ro;
        P.co = F.co;
        const int m = P.m, n = P.n;

        // A1: sign-normalise and classify rows; surplus columns by ballot.
        bool bad = F.bad_row;
        const bool gather = a.shared && a.row_subset;
        if (gather) {
#pragma unroll
            for (int r = 0; r < RB; ++r)
                if (lane + 64 * r < m) rowid[lane + 64 * r] = F.rid[r];
        }
        double bv[RB];
        int sc[RB];
        int ng = 0, nart = 0, neq = 0;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = lane + 64 * r;
            int f = kRowPad;
            const double bi = F.bv[r];
            if (i < m) {
                const int s = F.sv[r];
                bad |= !isfinite(bi) || s < kLE || s > kEQ;
                const bool neg = bi < 0.0;
                int sen = (s < kLE || s > kEQ) ? kLE : s;
                if (neg && sen != kEQ) sen = (sen == kLE) ? kGE : kLE;
                f = (neg ? kRowNeg : 0) | (sen << 1);
            }
            bv[r] = bi;
            P.rowf[r] = f;
            P.rhs[r] = (i < m) ? T((f & kRowNeg) ? -bi : bi) : T(0);
            const int sen = (f >> 1) & 3;
            const uint64_t ge = ballot(i < m && sen == kGE);
            const uint64_t ar = ballot(i < m && sen != kLE);
            const uint64_t eq = ballot(i < m && sen == kEQ);
            sc[r] = -1;
            if (i < m && sen == kGE) {
                const int g = ng + __popcll(ge & lanemask_lt(lane));
                sc[r] = n + g;
                if (g < 64 * RB) colrow[g] = i;
            }
            ng += __popcll(ge);
            nart += __popcll(ar);
            neq += __popcll(eq);
        }
        P.N = n + ng;
        P.C = P.N;
        P.ld = row_stride<T>(P.N);
        P.nart = nart;
        const int64_t need = aux + int64_t(m) * P.ld * int64_t(sizeof(T));
        const bool fits = P.C <= 64 && m <= 64 * RB && need <= a.lds_bytes;
        if (!fits && lane == 0) {
            const int slot = a.defer_base + atomicAdd(a.defer_count, 1);
            a.defer_ids[slot] = int32_t(k);
        }
        const int N = P.N, C = P.C, ld = P.ld;
        T *tab = reinterpret_cast<T *>(smem + aux);
        P.tab = tab;

#pragma unroll
        for (int r = 0; r < RB; ++r) P.rowat[r] = min(lane + 64 * r, m - 1) * ld;
        P.colat = min(lane, C - 1);

        // A2: index arrays and the tableau (row-major in LDS).
        wave_sync();  // colrow, rowid
        P.nonb = kBig;
        const double cj = fresh_copy(F.cv);
        if (fits) {
        if (lane < n) {
            P.nonb = lane;
            bad |= !isfinite(cj);
        } else if (lane < N) {
            P.nonb = n + colrow[lane - n];
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int i = lane + 64 * r;
            P.basis[r] = (((P.rowf[r] >> 1) & 3) == kLE) ? n + i : n + m + i;
        }
        {
            // A in flat row-major order, which is the tableau's own when its row
            // stride is n; otherwise element f = lane + 64 t, at row f / n and
            // column f % n, moves on by (f / n) (ld - n).  Stepping t by one
            // advances the column by 64 % n and the row by 64 / n, plus one
            // when the column wraps.
            const int mn = m * n;
            const int dq = 64 / n, dr = 64 - dq * n;
            int ri = lane / n, cj2 = lane - (lane / n) * n;
            if (PFD > 0 && F.has_a) {
                // Only the last, partial step needs a bounds test.  (Prefetched
                // elements past m * n read as 0, so every register can be checked
                // for finiteness.)
                const int full = mn >> 6;
#pragma unroll
                for (int t = 0; t < (PFD > 0 ? PFD : 1); ++t) bad |= !isfinite(F.av[t]);
                if (ld == n) {
                    T *at = tab + lane;
#pragma unroll
                    for (int t = 0; t < (PFD > 0 ? PFD : 1); ++t)
                        if (t < full || (t == full && lane + 64 * t < mn)) at[64 * t] = T(F.av[t]);
                } else {
                    const int gap = ld - n, step = 64 + gap * dq;
                    int pos = lane + gap * ri;
#pragma unroll
                    for (int t = 0; t < (PFD > 0 ? PFD : 1); ++t) {
                        if (t < full || (t == full && lane + 64 * t < mn)) tab[pos] = T(F.av[t]);
                        cj2 += dr;
                        pos += step;
                        if (cj2 >= n) { cj2 -= n; pos += gap; }
                    }
                }
            } else {
                // (Eight loads in flight for FP32 LPs of up to 64 rows, which have the
                // registers of five wavefronts per SIMD.)
                constexpr int UB = (sizeof(T) == 4 && RB == 1) ? 8 : 16;
                for (int f0 = 0; f0 < mn; f0 += 64 * UB) {
                    double av[UB];
                    if (gather) {
                        // Row f / n of the LP is constraint rowid[f / n] of the shared LP.
                        int rr = ri, cc = cj2;
#pragma unroll
                        for (int u = 0; u < UB; ++u) {
                            const int f = f0 + 64 * u + lane;
                            av[u] = 0.0;
                            if (f < mn) av[u] = P.A[int64_t(rowid[rr < m ? rr : m - 1]) * n + cc];
                            rr += dq;
                            cc += dr;
                            if (cc >= n) { cc -= n; ++rr; }
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < UB; ++u) {
                            const int f = f0 + 64 * u + lane;
                            av[u] = (f < mn) ? P.A[f] : 0.0;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < UB; ++u) {
                        if (f0 + 64 * u + lane < mn) {
                            bad |= !isfinite(av[u]);
                            tab[ri * ld + cj2] = T(av[u]);
                        }
                        ri += dq;
                        cj2 += dr;
                        if (cj2 >= n) { cj2 -= n; ++ri; }
                    }
                }
            }
            // Rows with b < 0 are negated (sign normalisation).
            wave_sync();
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                uint64_t neg = ballot(lane + 64 * r < m && (P.rowf[r] & kRowNeg));
                while (neg) {
                    const int i = 64 * r + __builtin_ctzll(neg);
                    neg &= neg - 1;
                    if (lane < n) tab[i * ld + lane] = -tab[i * ld + lane];
                }
            }
            // Surplus columns, one row per lane.
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int i = lane + 64 * r;
                if (i < m)
                    for (int g = 0; g < ng; ++g) tab[i * ld + n + g] = (sc[r] == n + g) ? T(-1) : T(0);
            }
        }
        wave_sync();
        }  // fits
        const double cnorm = wave_max_f(fabs(cj));
        double bm = 0.0;
#pragma unroll
        for (int r = 0; r < RB; ++r) bm = fmax(bm, fabs(bv[r]));
        const double bnorm = wave_max_f(bm);
        // The registers of F are free again: start loading the next LP.  (The
        // last one reloads itself, so the loads are unconditional and land in the
        // registers the current LP's came in.)
        fetch<RB, PFD>(nxt < total ? nxt : !STEEP && redo >= 0 ? redo : cur, F);
        if (!fits) {
            next_item();
            continue;
        }
        const bool invalid = ballot(bad) != 0;
        P.iters = 0; P.it1 = 0; P.degp = 0;
        P.alone = alone;
        P.cap = a.prm.max_iters > 0 ? a.prm.max_iters : 50 * (m + n + (m - neq) + nart);
        P.d = T(0);
        P.z = T(0);
        int status = kOptimal, enter = -1;

        // Warm start (repair instantiation): only from a relaxation that ended
        // optimal (its status is still in status[k]) with few violated rows,
        // and only for all-<= LPs; any other LP is solved from the slack basis
        // right here.  An LP whose repair fails is deferred.
        bool warm_ok = false, warm_defer = false;
        Pending<T, RB, NG> pend;  // warm start
        if (invalid) {
            status = kInvalid;
        } else {
            if constexpr (WARM) {
                warm_ok = nart == 0 && a.status[k] == kOptimal &&
                          !(a.warm_viol && a.warm_viol[k] > a.warm_max_viol);
                if (warm_ok) {
                    P.keep = true;
                    pend.clear();
                    warm_defer = !crash(P, pend, a, k) || overflowed(P);
                }
            }
            // Phase I where some row needs an artificial, then Phase II.
            for (int phase = nart > 0 ? 1 : 2; !warm_defer; phase = 2) {
                T eps_opt;
                int r = kPrimal;
                P.keep = phase == 1;
                if (phase == 1) {
                    // Objective row: sum of the artificial rows in row order.
                    T acc = T(0), zacc = T(0);
                    for (int i = 0; i < m; ++i) {
                        const int sen = (row_get<RB>(P.rowf, i) >> 1) & 3;
                        if (sen != kLE) {
                            if (lane < C) acc += tab[i * ld + lane];
                            zacc += row_get<RB>(P.rhs, i);
                        }
                    }
                    P.d = acc;
                    P.z = zacc;
                    const double dmax = wave_max_f(lane < N ? fabs(double(acc)) : 0.0);
                    eps_opt = T(a.prm.tol_opt * fmax(1.0, dmax));
                } else {
                    // Objective row: c priced out over the basis, rows in order.
                    T cb[RB];
                    uint64_t nz[RB];
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        const int bvr = P.basis[r];
                        const double cbv = __shfl(cj, bvr < n ? bvr : 0);  // c of the row's basic variable
                        cb[r] = (!(P.rowf[r] & (kRowDead | kRowPad)) && bvr < n) ? T(cbv) : T(0);
                        nz[r] = ballot(cb[r] != T(0));
                    }
                    const double cnb = __shfl(cj, (P.nonb >= 0 && P.nonb < n) ? P.nonb : 0);
                    T acc = (lane < N && P.nonb < n) ? T(cnb) : T(0), zacc = T(0);
#pragma unroll
                    for (int r = 0; r < RB; ++r) {
                        uint64_t mk = nz[r];
                        while (mk) {
                            const int bit = __builtin_ctzll(mk);
                            mk &= mk - 1;
                            const T f = lane_get(cb[r], bit);
                            if (lane < C) acc = fma(-f, tab[(64 * r + bit) * ld + lane], acc);
                            zacc = fma(-f, lane_get(P.rhs[r], bit), zacc);
                        }
                    }
                    P.d = acc;
                    P.z = zacc;
                    eps_opt = T(a.prm.tol_opt * fmax(1.0, cnorm));
                    // Single-precision level for the start's reduced costs.
                    if (WARM && warm_ok)
                        r = dual_repair(P, pend, T(1e-5 * fmax(1.0, cnorm)), T(a.prm.tol_feas * (1.0 + bnorm)), a.prm);
                }
                if (r == kPrimal) r = simplex<STEEP, T, RB, NG>(P, eps_opt, a.prm, &enter);
                if (WARM && r == kAgain) {
                    warm_defer = true;
                    break;
                }
                if (phase == 2) {
                    status = r;
                    if (WARM && warm_ok) warm_defer = status != kOptimal;
                    break;
                }
                P.it1 = P.iters;
                enter = -1;
                if (r == kIterLimit) status = kIterLimit;
                else if (r == kUnbounded) status = kNumerical;
                else if (r == kAgain) status = kAgain;
                else if (-double(P.z) < -a.prm.tol_feas * (1.0 + bnorm)) status = kInfeasible;
                if (status != kOptimal) break;
                // Drive basic artificials out in row order; drop redundant rows.
                const T tol_piv = T(a.prm.tol_piv);
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    uint64_t am = ballot(lane + 64 * r < m && P.basis[r] >= n + m);
                    while (am) {
                        const int bit = __builtin_ctzll(am);
                        am &= am - 1;
                        const int i = 64 * r + bit;
                        bool ok = false;
                        if (lane < N && P.nonb < n + m) ok = fabs(tab[i * ld + lane]) > tol_piv;
                        const int e = price<T>(ok, T(0), P.nonb, true);
                        if (e >= 0) {
#pragma unroll
                            for (int q = 0; q < RB; ++q)
                                P.pcol[q] = P.rowf[q] & (kRowDead | kRowPad) ? T(0) : tab[P.rowat[q] + e];
                            const T rowv = tab[i * ld + P.colat];
                            replace(P, i, e, scaled_row(P, i, e, rowv),
                                    row_get<RB>(P.rhs, i) / row_get<RB>(P.pcol, i));
                        } else if (lane == bit) {
                            P.rowf[r] |= kRowDead;
                        }
                    }
                }
            }
        }
        if (WARM && warm_defer) {
            if (lane == 0) {
                // Not optimal any more: the workgroup kernel that drains the
                // deferred list then solves it from the slack basis.
                a.status[k] = kNumerical;
                const int slot = a.defer_base + atomicAdd(a.defer_count, 1);
                a.defer_ids[slot] = int32_t(k);
            }
            next_item();
            continue;
        }

        // A8: extraction through an LDS staging vector.
        const auto &out = *late_args();
        // The tableau is free now: x is staged in its place.
        T *xv = tab;
        wave_sync();
        if (lane < n) xv[lane] = T(0);
        wave_sync();
        if (status == kOptimal) {
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int i = lane + 64 * r;
                const int bvr = P.basis[r];
                if (i < m && bvr < n && !(P.rowf[r] & kRowDead)) xv[bvr] = P.rhs[r];
            }
        }
        wave_sync();
        const double xj = (lane < n) ? double(xv[lane]) : 0.0;
        if (lane < n) out.x[P.co + lane] = (status == kOptimal) ? xj : __builtin_nan("");
        double z = (lane < n) ? fma(cj, xj, 0.0) : 0.0;
        int nbs = (lane < n && xj != 0.0) ? 1 : 0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            z += __shfl_xor(z, off);
            nbs += __shfl_xor(nbs, off);
        }
        if (lane == 0) {
            double objv = z;
            if (status == kUnbounded) objv = __builtin_inf();
            else if (status != kOptimal) objv = __builtin_nan("");
            out.obj[k] = objv;
            out.status[k] = status;
            if (out.enter_out) out.enter_out[k] = (status == kUnbounded) ? enter : -1;
            if (out.stats) {
                int32_t *st = out.stats + 8 * k;
                if (out.refine_stats) {
                    st[3] = warm_ok ? 2 : 1;  // 2: started from the relaxation's basis
                    st[4] = P.iters;
                } else {
                    st[0] = P.it1;
                    st[1] = P.iters - P.it1;
                    st[2] = P.degp;
                    st[3] = 0;
                    st[4] = 0;
                    st[5] = 0;
                }
                st[6] = 1;
                st[7] = nbs;
            }
        }
        if (out.basis_out) {
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int i = lane + 64 * r;
                if (i < m) out.basis_out[P.ro + i] = (P.rowf[r] & kRowDead) ? -1 : P.basis[r];
            }
        }
        if (!STEEP && uniform(status) == kAgain) {
            // Onto the list; the last LP of all is in F already.
            if (nxt >= total && redo < 0) {
                alone = 1;
                continue;
            }
            const int was = int(cur);
            next_item();
            if (lane == 0) *const_cast<volatile int32_t *>(a.status + P.k) = redo;
            redo = was;
            continue;
        }
        next_item();
    }
    drain_memory();
    if (lane == 0) finish_launch(a.queue, a.reset_extra);
}


template <typename T, int RB, int PFD, bool WARM = false, bool STEEP = false>
hipError_t launch_t(const SolveArgs &a, int grid, hipStream_t s)
{
    hipLaunchKernelGGL((simplex_wave_kernel<T, RB, PFD, WARM, STEEP>), dim3(grid), dim3(64), a.lds_bytes, s, a);
    return hipGetLastError();
}

template <typename T, int RB, int PFD, bool WARM = false, bool STEEP = false>
int occ_t(int lds)
{
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, (const void *)simplex_wave_kernel<T, RB, PFD, WARM, STEEP>, 64, lds) != hipSuccess)
        return 0;
    return blocks;
}

template <typename T>
hipError_t launch_rb(int rb, bool pf, const SolveArgs &a, int grid, hipStream_t s)
{
    if (a.prm.pricing == 1)
        return rb == 1 ? launch_t<T, 1, 0, false, true>(a, grid, s)
             : rb == 2 ? launch_t<T, 2, 0, false, true>(a, grid, s) : hipErrorInvalidValue;
    if (rb == 1) return pf ? launch_t<T, 1, NPF>(a, grid, s) : launch_t<T, 1, 0>(a, grid, s);
    return rb == 2 && !pf ? launch_t<T, 2, 0>(a, grid, s) : hipErrorInvalidValue;
}

template <typename T>
int occ_rb(int rb, bool pf, bool steep, int lds)
{
    if (steep) return rb == 1 ? occ_t<T, 1, 0, false, true>(lds) : rb == 2 ? occ_t<T, 2, 0, false, true>(lds) : 0;
    if (rb == 1) return pf ? occ_t<T, 1, NPF>(lds) : occ_t<T, 1, 0>(lds);
    return rb == 2 && !pf ? occ_t<T, 2, 0>(lds) : 0;
}

}  // namespace

int64_t wave_lds_aux_bytes(int rb, bool gather) { return wave_aux_bytes(rb, gather); }

int64_t wave_tab_bytes(int m, int cols, bool fp32)
{
    return fp32 ? int64_t(m) * row_stride<float>(cols) * 4 : int64_t(m) * row_stride<double>(cols) * 8;
}

int wave_prefetch_elems() { return 64 * NPF; }

hipError_t launch_simplex_wave(bool fp32, int rb, bool pf, const SolveArgs &a, int grid, hipStream_t s)
{
    return fp32 ? launch_rb<float>(rb, pf, a, grid, s) : launch_rb<double>(rb, pf, a, grid, s);
}

int simplex_wave_blocks_per_cu(bool fp32, int rb, bool pf, bool steep, int lds)
{
    return fp32 ? occ_rb<float>(rb, pf, steep, lds) : occ_rb<double>(rb, pf, steep, lds);
}

hipError_t launch_simplex_wave_warm(int rb, const SolveArgs &a, int grid, hipStream_t s)
{
    if (!a.warm_basis || (a.warm_rows && a.warm_m < 1)) return hipErrorInvalidValue;
    const bool steep = a.prm.pricing == 1;
    if (rb == 1) return steep ? launch_t<double, 1, 0, true, true>(a, grid, s) : launch_t<double, 1, 0, true>(a, grid, s);
    if (rb == 2) return steep ? launch_t<double, 2, 0, true, true>(a, grid, s) : launch_t<double, 2, 0, true>(a, grid, s);
    return hipErrorInvalidValue;
}

int simplex_wave_warm_blocks_per_cu(int rb, bool steep, int lds)
{
    if (rb == 1) return steep ? occ_t<double, 1, 0, true, true>(lds) : occ_t<double, 1, 0, true>(lds);
    if (rb == 2) return steep ? occ_t<double, 2, 0, true, true>(lds) : occ_t<double, 2, 0, true>(lds);
    return 0;
}

hipError_t simplex_wave_configure(int max_lds)
{
    const void *fns[] = {(const void *)simplex_wave_kernel<float, 1, NPF>, (const void *)simplex_wave_kernel<double, 1, NPF>,
                         (const void *)simplex_wave_kernel<float, 1, 0>,   (const void *)simplex_wave_kernel<double, 1, 0>,
                         (const void *)simplex_wave_kernel<float, 2, 0>,   (const void *)simplex_wave_kernel<double, 2, 0>,
                         (const void *)simplex_wave_kernel<float, 1, 0, false, true>,
                         (const void *)simplex_wave_kernel<double, 1, 0, false, true>,
                         (const void *)simplex_wave_kernel<float, 2, 0, false, true>,
                         (const void *)simplex_wave_kernel<double, 2, 0, false, true>,
                         (const void *)simplex_wave_kernel<double, 1, 0, true>,
                         (const void *)simplex_wave_kernel<double, 2, 0, true>,
                         (const void *)simplex_wave_kernel<double, 1, 0, true, true>,
                         (const void *)simplex_wave_kernel<double, 2, 0, true, true>};
    for (const void *f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lpb
