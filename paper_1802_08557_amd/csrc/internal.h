// internal.h -- structures shared by the host runtime and the HIP kernels.
// Not part of the public ABI (include/lpbatch.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lpb {

__host__ __device__ inline int64_t align16(int64_t v) { return (v + 15) & ~int64_t(15); }

// Tolerances and limits of one solve (the public lp_options with defaults filled in).
struct SolveParams {
    double tol_piv;    // a pivot-column entry must exceed this to be eligible (Step 2)
    double tol_opt;    // reduced costs above tol_opt * max(1, |c|_inf) may enter (Step 1)
    double tol_feas;   // Phase I optimum below -tol_feas * (1 + |b|_inf) means infeasible
    int32_t k_deg;     // consecutive degenerate pivots before Bland's rule; <= 0: never
    int32_t max_iters; // pivot cap over both phases; <= 0: 50 * (m + #columns)
    int32_t pricing;   // 0: Dantzig; 1: steepest edge (d_j^2 / (1 + |column j|^2))
};

// The work queue of one launch: kQueues counters, each in a cache line of its
// own, and per counter the workgroups that have finished (all 0 between
// launches).  Worker b of the launch pops from counter b % kQueues, which hands
// out the items congruent to it.  Atomics on one address take 12 ns each on
// MI355X whatever the kernel around them does, so a single counter held every
// launch over small LPs to 12 ns per LP -- 1.2 ms per 1e5 -- plus 12 ns per
// workgroup at its end.
constexpr int kQueues = 16;
constexpr int kQueueLine = 32;                              // int32 per line
constexpr int kQueueInts = (kQueues + 1) * kQueueLine;      // the last line counts finished counters

// Everything one launch of the simplex kernel needs.  Device pointers unless noted.
struct SolveArgs {
    int64_t num;              // work items in this launch (upper bound if num_dev is set)
    const int32_t *ids;       // work item -> LP index; null: identity
    const int32_t *num_dev;   // optional device-side count: items = id_base + *num_dev
    int32_t id_base;
    const double *A, *b, *c;  // batch data, layout of include/lpbatch.h
    const int8_t *sense;
    int32_t um, un;           // > 0: every LP is um x un (offsets computed, m/n/offsets unused)
    int32_t shared;           // 1: A, b, sense hold one LP of m_full x un shared by all LPs
                              //   (c, x, status, obj and basis_out stay per LP)
    const int32_t *row_subset;// shared only, optional [num][um]: LP k's row r is row
    int32_t m_full;           //   row_subset[k*um + r] of the shared LP (um <= m_full);
                              //   an index outside [0, m_full) makes the LP INVALID_INPUT
    const int32_t *m, *n;     // per-LP sizes when not uniform
    const int64_t *aoff, *roff, *coff;
    int32_t *status;          // outputs
    double *x, *obj;
    int32_t *stats;           // optional [num_lps][8]
    int32_t *basis_out;       // optional [sum m]: final basis (Bland index, -1 dropped row)
    int32_t *enter_out;       // optional [num_lps]: entering Bland index at UNBOUNDED
    char *scratch;            // HBM tableau slots, one per workgroup of the launch
    int64_t slot_bytes;
    int32_t *queue;           // kQueueInts work counters (0 at launch); the last workgroup to
                              // finish resets them and reset_extra to 0 for the next launch.
                              // NULL: the grid has a worker for every item
    int32_t *reset_extra;     // optional
    int32_t *defer_ids;       // wavefront kernel: LPs it could not take are appended here,
    int32_t *defer_count;     //   from defer_ids[defer_base] on (the workgroup kernel
    int32_t defer_base;       //   then drains them)
    int32_t lds_bytes;        // dynamic LDS of each workgroup
    int32_t least_window;     // workgroup kernel: pivots that the window beside a tableau in LDS
                              // must hold (>= kLeastWindow), or it goes to device memory
    int32_t force_hbm;        // 1: never keep the tableau in LDS
    int32_t refine_stats;     // 1: a re-solve -- pivots go to stats[4], stats[3] = 1
    // Warm start of a re-solve (wavefront kernel, FP64, all-<= LPs): LP k
    // starts from the final basis of a relaxation solved on warm_m of its rows
    // -- warm_basis[k*warm_m + r] is the Bland index (relaxation numbering) of
    // the variable basic in relaxation row r, which is row warm_rows[k*warm_m + r]
    // of the LP.  Structurals are pivoted in, then the dual simplex method
    // repairs primal feasibility; an LP the repair does not finish optimal is
    // deferred to the workgroup kernel, which solves it from the slack basis.
    const int32_t *warm_basis;
    const int32_t *warm_rows;
    int32_t warm_m;
    const int32_t *warm_viol; // optional [num]: rows the relaxation's optimum violates; more
    int32_t warm_max_viol;    //   than warm_max_viol sends the LP to the slack-basis solve
    SolveParams prm;
};

// One launch of the FP64 certificate kernel (certify_kernels.hip).
struct CertArgs {
    int64_t num;
    const double *A, *b, *c;
    const int8_t *sense;
    int32_t um, un;
    int32_t shared;           // as in SolveArgs (um = rows of the shared LP)
    const int32_t *row_subset;// optional: the basis came from a solve on these rows only,
    int32_t subset_m;         //   subset_m per LP (basis and enter use that LP's numbering)
    const int32_t *m, *n;
    const int64_t *aoff, *roff, *coff;
    int32_t *status;
    double *x, *obj;
    int32_t *stats;
    const int32_t *basis;     // final basis of the single-precision solve
    const int32_t *enter;     // entering variable at UNBOUNDED
    int32_t *fb_ids;          // LPs to re-solve in FP64 are appended here
    int32_t *fb_count;
    int32_t *viol;            // optional [num]: rows the basis's x violates (wavefront kernel)
    char *scratch;            // LU matrices too large for LDS, one slot per workgroup
    int64_t slot_bytes;
    int32_t *queue;           // as in SolveArgs
    // Workgroup kernel, optional: work item t is LP order1[t] for t < n1, else
    // order2[t - n1] (largest LPs first, so the launch does not end on one);
    // NULL: item t is LP t.
    const int32_t *order1, *order2;
    int64_t n1;
    int32_t lds_bytes;
    double tol_feas, tol_opt; // certificate tolerances (relative, as in SolveParams)
    // Wavefront kernels only: LDS bytes per wavefront (the dense kernel: the
    // bytes of its staged A), LU blocks up to kl x kl kept in LDS (a larger
    // basis goes to the FP64 re-solve), and whether the shared constraint
    // matrix is copied into LDS.
    int32_t wave_bytes, kl, stage_a;
};

// LDS carve-up of one LP in the wavefront certificate kernel (byte offsets).
struct WaveCertLayout {
    int64_t rowf, tpos, colf, spos, tlist, slist, order, xs, yv, mat, end;
};

__host__ __device__ inline WaveCertLayout wave_cert_layout(int m, int n, int kl)
{
    WaveCertLayout L;
    int64_t o = 0;
    L.rowf = o; o = align16(o + 4 * int64_t(m));
    L.tpos = o; o = align16(o + 4 * int64_t(m));
    L.colf = o; o = align16(o + 4 * int64_t(n));
    L.spos = o; o = align16(o + 4 * int64_t(n));
    L.tlist = o; o += 256;
    L.slist = o; o += 256;
    L.order = o; o += 256;
    L.xs = o; o = align16(o + 8 * int64_t(kl));  // x_S and y_T: k <= kl entries
    L.yv = o; o = align16(o + 8 * int64_t(kl));
    L.mat = o; o = align16(o + 8 * int64_t(kl) * (kl | 1));  // column stride k | 1
    L.end = o;
    return L;
}

hipError_t launch_certify_wave(int waves, const CertArgs &a, int grid, hipStream_t s);
int certify_wave_blocks_per_cu(int waves, int lds_bytes);

// Dense certificate (certify_dense.hip): one wavefront per LP of at most 64 x
// 64 and certify_dense_prefetch_elems() entries, own A (not shared, not
// screened); wave_bytes = certify_dense_a_bytes(m_max, n_max), kl <= 64.
hipError_t launch_certify_dense(const CertArgs &a, int grid, hipStream_t s);
int certify_dense_blocks_per_cu(int lds_bytes);
int64_t certify_dense_a_bytes(int m_max, int n_max);
int64_t certify_dense_lds_bytes(int m_max, int n_max, int kl);
int certify_dense_prefetch_elems();
hipError_t certify_dense_configure(int max_lds);

hipError_t launch_certify(int nt, const CertArgs &a, int grid, hipStream_t s);
int certify_blocks_per_cu(int nt, int lds_bytes);
int64_t certify_lds_bytes(int m, int n, bool with_matrix);
hipError_t certify_configure(int max_lds);

// Warm-start network (mlp_kernels.hip).  The gradients of B labelled rows: FP32
// parameters w32 and their BF16 copy w16 in, grad [LP_MLP_NUM_PARAMS] and
// loss[0] out; the rest is scratch: dS, dZ2, dZ1 and the row losses in FP32
// ([B][...]), and the BF16 operands of the dW products transposed, [columns][ldt]
// with ldt >= B rounded up to 16.
struct MlpTrain {
    int64_t B, ldt;
    const float *dirs, *w32;
    const uint8_t *tight;
    const uint16_t *w16;
    float *ds, *dz2, *dz1, *row_loss;
    uint16_t *xt, *h1t, *h2t, *dst, *dz2t, *dz1t;
    float *grad, *loss;
};
hipError_t launch_mlp_grads(const MlpTrain &g, hipStream_t s);

struct MlpAdam {
    float lr, wd, beta1, beta2, eps, bc1, bc2;  // bc = 1 - beta^t
};

hipError_t launch_adamw(float *w, const float *g, float *m, float *v, uint16_t *w16, int64_t count,
                        const MlpAdam &h, const int64_t (&decay)[6], hipStream_t s);
hipError_t launch_cast_params(const float *w, uint16_t *w16, int64_t count, hipStream_t s);
// Fused inference (all layers and the top-k, tiles of 64 directions):
// scores [B][120] and/or topk [B][k] (either may be NULL).
hipError_t launch_mlp_infer(const float *dirs, int64_t B, const uint16_t *w16, const float *w32, float *scores,
                            int32_t *topk, int k, hipStream_t s);
hipError_t mlp_configure();

// Closed-form box LPs (hyperbox_kernels.hip).
hipError_t launch_hyperbox(int64_t num, int n, const double *lo, const double *hi, const double *l,
                           int shared_box, double *value, double *x, hipStream_t s);

// Power-of-two scaling (scale_kernels.hip).  um/un: uniform shape, or 0 with
// the per-LP shape and offset arrays; c_out may be NULL (c left alone).
// host_m / host_n: the shapes in host memory (read to size the launch).
hipError_t launch_scale(int64_t num, int32_t um, int32_t un, const int32_t *m, const int32_t *n,
                        const int64_t *aoff, const int64_t *roff, const int64_t *coff, const int32_t *host_m,
                        const int32_t *host_n, int32_t passes, const double *A, const double *b, const double *c,
                        double *A_out, double *b_out, double *c_out, int32_t *rexp, int32_t *cexp, hipStream_t s);
// out[i] = in[i] * 2^e[i] (period 0) or 2^e[i % period]; in may equal out.
hipError_t launch_ldexp(int64_t count, const double *in, const int32_t *e, int64_t period, double *out,
                        hipStream_t s);

// Bland index convention shared by every kernel: structural j -> j, the
// slack/surplus of row i -> n + i, the artificial of row i -> n + m + i.

// Statically allocated device scratch of lp_batch_solve_noalloc (noalloc.hip):
// 8 KiB of work counters, the deferred-LP list (kNoAllocMaxLps entries),
// then the workgroup kernel's tableau slots.
constexpr int64_t kNoAllocBytes = int64_t(16) << 20;
constexpr int64_t kNoAllocMaxLps = int64_t(1) << 20;
constexpr int64_t kNoAllocIdsAt = 8192;
constexpr int64_t kNoAllocSlotsAt = kNoAllocIdsAt + 4 * kNoAllocMaxLps;
// Device address of this device's copy (the current device's).
hipError_t noalloc_scratch_address(void **ptr);

// Launchers (simplex_kernels.hip).  Return the hipError_t of the launch.
hipError_t launch_zero_i32(int32_t *p, int count, hipStream_t s);
hipError_t launch_simplex(bool fp32, int nt, const SolveArgs &a, int grid, hipStream_t s);
// Workgroups of the simplex kernel that fit one CU with this LDS (occupancy query).
int simplex_blocks_per_cu(bool fp32, int nt, int lds_bytes);
// Bytes of the kernel's LDS control block for the given tableau precision.
int64_t simplex_ctrl_bytes(bool fp32);
// Allows every simplex kernel instantiation up to max_lds bytes of dynamic LDS.
hipError_t simplex_configure(int max_lds);

// One-wavefront-per-LP kernel (wave_kernels.hip) for LPs of at most 64
// non-basic columns and 64*rb rows (rb = 1 or 2).
// pf: the instantiation that prefetches each next LP's A into registers
// (rb = 1, LPs of at most wave_prefetch_elems() entries, A not row-gathered).
hipError_t launch_simplex_wave(bool fp32, int rb, bool pf, const SolveArgs &a, int grid, hipStream_t s);
// The warm-start (repair) instantiation: FP64, no prefetch; a.warm_basis set.
hipError_t launch_simplex_wave_warm(int rb, const SolveArgs &a, int grid, hipStream_t s);
int simplex_wave_warm_blocks_per_cu(int rb, bool steep, int lds_bytes);
int simplex_wave_blocks_per_cu(bool fp32, int rb, bool pf, bool steep, int lds_bytes);
int wave_prefetch_elems();
int64_t wave_lds_aux_bytes(int rb, bool gather);
// LDS bytes of a wavefront tableau with m rows and `cols` columns.
int64_t wave_tab_bytes(int m, int cols, bool fp32);
hipError_t simplex_wave_configure(int max_lds);

// Rows up to which the workgroup kernel updates a tableau in LDS pivot by pivot
// instead of through a window of deferred pivots.
constexpr int kDirectRows = 12;

// The least window (pivots) that the workgroup kernel asks for beside its arrays.
constexpr int kLeastWindow = 2;

// LDS of the workgroup kernel for an LP of m rows and N non-basic columns (byte
// offsets): control block, index arrays, right-hand sides, reduced costs, then
// the window of deferred pivots (a column of m and a row of N entries each),
// then, where it fits, the tableau.  The offsets up to rhs do not depend on N.
struct LdsLayout {
    int64_t basis, rowf, colrow, rhs, nonb, obj, win, vec;
    // End of a window of K pivots: where an LDS-resident tableau starts.
    __host__ __device__ int64_t window(int64_t K) const { return align16(win + K * vec); }
};

// ctrl_bytes: size of the control block (type dependent, passed by the caller).
__host__ __device__ inline LdsLayout lds_layout(int m, int N, int64_t tsize, int64_t ctrl_bytes)
{
    LdsLayout L;
    L.basis = align16(ctrl_bytes);
    L.rowf = L.basis + 4 * int64_t(m);
    L.colrow = L.rowf + 4 * int64_t(m);
    L.rhs = align16(L.colrow + 4 * int64_t(m));
    L.nonb = align16(L.rhs + tsize * int64_t(m));
    L.obj = align16(L.nonb + 4 * int64_t(N));
    L.win = align16(L.obj + tsize * int64_t(N));
    L.vec = tsize * (int64_t(m) + N);
    return L;
}

// Row stride (elements) of a workgroup-kernel tableau of N columns.  In LDS: no
// multiple of four, so that walking a column spreads over the banks; in device
// memory: whole cache lines of 128 bytes.
__host__ __device__ inline int lds_tab_ld(int N) { return N & 3 ? N : N + 1; }
__host__ __device__ inline int64_t lds_tab_bytes(int m, int N, int tsize)
{
    return int64_t(tsize) * m * lds_tab_ld(N);
}
__host__ __device__ inline int slot_tab_ld(int N, int tsize)
{
    const int R = 128 / tsize;
    return (N + R - 1) / R * R;
}

}  // namespace lpb
