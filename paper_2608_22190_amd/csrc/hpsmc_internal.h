// Internal declarations shared by the host runtime (hpsmc_host.cpp) and the
// gfx950 kernels (hpsmc_kernels.hip).  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace hpsmc {

constexpr int kMaxDim = 5;
constexpr int kMaxN = 32;            // spatial nodes per dimension
constexpr int kMaxP = kMaxN + 2;     // Legendre modes per dimension (phi_p has degree p+2)
constexpr int kMaxDeg = 31;          // temporal degree M_n

// One Monte Carlo node (instance, interval, l >= 1, spatial node j).
struct NodeDesc {
    double x0[kMaxDim];   // spatial node
    double delta;         // Delta_{n,l} = (t_{n,l} - t_{n-1}) / N*
    double jump;          // J = sqrt(2 d Delta)
    double span;          // t_{n,l} - t_{n-1}
    double t_prev;        // t_{n-1}
    int64_t u_index;      // offset of U[inst][iv][j][l] in the nodal buffer
    int64_t slab;         // offset of the q = 0 slab of (inst, iv, l) in the slab table
    int32_t nstar;        // N*
    uint32_t c0;          // Philox counter word 0: j + n^d (l - 1)
    uint32_t c3;          // Philox counter word 3 without the tag: inst<<16 | iv<<8
    int32_t out;          // row of this node in the per-launch output arrays
};

// One (instance, interval, l) group: its nodes share the slab sequence, N*,
// Delta and J, so a block can advance any mix of their paths in lockstep.
struct GroupDesc {
    double delta, jump, span, t_prev;
    int64_t slab;          // offset of the q = 0 slab in the slab table (row layout)
    int64_t slab_mma;      // the same in the matrix-core layout (d = 2, FP32)
    int64_t path_off;      // first path slot of the group in the state buffers
    int32_t nstar;
    int32_t node_begin;    // the group's nodes are [node_begin, node_begin + node_count)
    int32_t node_count;
    uint32_t c3;           // Philox counter word 3 without the tag
    int32_t blk;           // the set's coefficient block of the group's (interval, instance)
};

// intervals of the tables of the fractional walk's inverse incomplete beta (a cubic each)
constexpr int kFracTab = 256;
constexpr int kFracTerms = 60;   // series terms of its Newton step in FP64

// The device's counters: the round's work counter, then the statistics in stripes of a
// cache line.  Every wave adds to its block's stripe: atomics on one line, from all the
// chip's waves, are served one by one (8192 of them held a launch of 1024 blocks for
// 55 us).
constexpr int kStatStripes = 64, kStatWords = 16;
constexpr int kCounterWords = kStatWords * (1 + kStatStripes);

// Problem constants every sampling lane needs.
struct Physics {
    int32_t dim, f_kind, src_kind;
    int32_t picard;              // 1: Picard-form estimator (eq. uast)
    int32_t ball;                // 1: integrand at the step's Green's-function ball point
    int32_t frac;                // 1: fractional operator (d = 1, alpha-stable walk)
    int32_t frac_kmax, frac_nt;  // recurrence length (a multiple of 4), series terms of the inverse
    int32_t frac_P;              // Jacobi modes of the slab
    double frac_a;               // alpha / 2
    double frac_half;            // I_{1/2}(a, 1 - a): the branch of the inverse
    double frac_lpb1, frac_lpb2; // log(a B(a, 1-a)), log((1-a) B(1-a, a))
    double frac_xs[2];           // kFracTab / X0max per branch
    const void *frac_tab;        // in the sampling precision: A, C, lambda, src [kmax each], cubics [2][kFracTab][4],
                                 // ra[nt], rb[nt]
    double f_param[4];
    double src_param[8];
};

// Arguments of the persistent sampling kernel.
struct SampleArgs {
    const NodeDesc *nodes;       // all nodes of this launch, in scheduling order
    int64_t n_nodes;
    int64_t M;                   // samples per node
    int32_t chunks_per_node;     // ceil(M / (64 * samples_per_lane))
    int32_t P;                   // Legendre modes per dimension
    int32_t PP;                  // padded row length of the slab (>= P, multiple of 4)
    int32_t tag;                 // iteration / sweep tag of the counter
    uint32_t key0, key1;
    const void *slab_table;      // T, rows of [u: PP][v: PP]
    int64_t slab_stride;         // elements per (inst, iv, l, q) slab
    double *part;                // [node out][chunk][2]: sum S, sum S^2
    double *probe;               // [node out][m_probe] or null
    int64_t m_probe;
    unsigned long long *work;    // work-item counter (zeroed before launch)
    unsigned long long *stats;   // [kStatStripes][kStatWords]: [0] residual evaluations, [1] lane steps
    Physics phys;
};

// Arguments of one round of the path-advancing kernel: every live path of
// every group advances by up to `steps` walk steps, the survivors are
// compacted into the other state buffer.
struct RoundArgs {
    const GroupDesc *groups;
    const NodeDesc *nodes;
    int32_t n_groups;
    int32_t round, steps;        // steps [round*steps, (round+1)*steps)
    int32_t batch;               // paths per block work item (64 * waves * NS)
    int64_t m0, mcount;          // sample slice [m0, m0 + mcount)
    const void *state_in;
    void *state_out;
    const uint32_t *live_in;     // per group, paths in state_in (round > 0)
    uint32_t *live_out;          // per group, survivors appended to state_out
    const int64_t *batch_prefix; // [n_groups + 3] batches per group, prefix ([n_groups]: work items, batches
                                 // times shares); [n_groups + 1] paths per batch; [n_groups + 2] shares
    double *share_val;           // [batch][window of the round, then the end][path of the batch] sums
    int32_t share_rows;          // windows of the round and one
    uint32_t *share_done;        // [batch] shares that have written theirs
    double *result;              // [node out][mcount] path value S of each sample
    int32_t n_chunks;            // LDS chunks per slab: P^cf, the first cf dimensions fixed per chunk
    int32_t cf;
    int64_t chunk_elems;         // slab elements per chunk (P^{d-1-cf} rows)
    int32_t P, PP, tag;
    uint32_t key0, key1;
    const void *slab_table;
    int64_t slab_stride;
    const float *inv_scale;      // matrix-core images of scaled coefficients: [blk][u, v] the inverse scale
    float bscale;                // the scale of their basis values
    int32_t mma_split;           // 2-D matrix-core kernel: products of halves
    unsigned long long *work;    // block work counter (zeroed by the prep kernel)
    unsigned long long *stats;   // [kStatStripes][kStatWords]: [0] residual evaluations, [1] slot steps
    Physics phys;
};

// One-dimensional lattice form: the points x_j + (mlo + i) J, i < 2 W, cover
// (-1, 1); the table of a round holds W entries (those of the step's parity) per
// node and step, [node][step][W].
struct LatDesc {
    int64_t toff;          // sum of W over the nodes before
    int32_t mlo, W;        // W even
};
struct LatArgs {
    const LatDesc *desc;   // per node
    double *table;
    const GroupDesc *groups;   // whose nodes they are
    int32_t n_groups, emax;    // most entries of a group's step
    int32_t win, wmax;         // steps per LDS window, widest W
};

// Arguments of one round of the adjoint kernel: the forward paths of one
// iteration are regenerated and every residual evaluation scatters its
// weighted basis values into the slab-adjoint table.
struct AdjointArgs {
    RoundArgs r;                 // paths, slabs, counters (result unused)
    const double *lambda;        // nodal adjoint, U layout
    void *slab_bar;              // slab-adjoint table, slab layout, type T
    double inv_M;                // 1/M
    int32_t use_mfma;            // FP32 only: 1 outer products on the matrix cores; 2 (d = 2) u* too, from
                                 // the slabs in the matrix-core layout (r.slab_stride, GroupDesc::slab_mma)
    int64_t bar_stride;          // elements per step of the slab-adjoint table (row layout, GroupDesc::slab)
};

// Time contraction of the modal coefficients into per-step spatial slabs.
// One group = one (instance, interval, node time l).
struct SlabArgs {
    const double *cu, *cv;       // Legendre tensors, blocks of [P^d][T1]
    const double *cs;            // polynomial source, blocks of [P^d][T1] per interval (null: none);
                                 // added to v in the contraction
    const int64_t *cs_off;       // per group: offset of its interval's source block
    const int64_t *coef_off;     // per group: offset of its (inst, iv) coefficient block
    const int64_t *slab_off;     // per group: offset of its q = 0 slab in the table (row layout)
    const int64_t *slab_off_mma; // the same in the matrix-core layout (null when not available)
    int64_t mma_stride;          // elements per slab in the matrix-core layout
    const int32_t *blk;          // per group: its coefficient block
    const int32_t *blk_group;    // per coefficient block: its first group
    int32_t n_blk;
    double *scale_max;           // [blk][u, v][scale_parts] largest entries over the parts of the block
    int32_t scale_parts;
    float *inv_scale;            // [blk][u, v] 1 / (scale bscale)
    double *pack;                // images of halves: [blk][pack_t][mma_stride] scaled coefficients in image order
    int32_t pack_t;              // most time coefficients of a block
    double bscale;
    int32_t split;               // the matrix-core layout holds halves
    int32_t layout;              // 0: rows [k0][u: PP][v: PP]; 1: matrix-core layout
    int32_t extra;               // slabs past N* per group (1 for the Picard form: q = N*, t_{n-1})
    const double *span;          // per group: t_{n,l} - t_{n-1}
    const double *delta;         // per group: Delta_{n,l}
    const double *h2;            // per group: 2 / h_n
    const int32_t *nstar;        // per group: N*
    const int32_t *deg;          // per group: M_n
    int32_t n_groups;
    int32_t P, PP, rows;         // rows = P^{d-1}
    int64_t slab_stride;         // rows * 2 * PP
    void *slab_table;
};

// Launch wrappers (hpsmc_kernels.hip).
hipError_t launch_mode_product(const double *in, double *out, int64_t outer, int len_in, int len_out,
                               int64_t inner, const double *mat, double alpha, int accumulate,
                               hipStream_t s);
hipError_t launch_slabs(const SlabArgs &a, int fp32, int max_nstar, hipStream_t s);
hipError_t launch_coef_pack(const SlabArgs &a, hipStream_t s);
hipError_t launch_sample(const SampleArgs &a, int fp32, int samples_per_lane, int waves_per_block,
                         int blocks, hipStream_t s);
hipError_t launch_reduce_update(const double *part, int chunks, int mode, const NodeDesc *nodes, int64_t n_nodes,
                                int64_t M, double *U, double *eps, double *sumsq,
                                unsigned long long *maxbits, hipStream_t s);
// Aitken-relaxed update of the vectors [vbeg[v], vbeg[v+1]) of a node set
hipError_t launch_aitken(const NodeDesc *nodes, const int64_t *vbeg, int n_vec, const double *eps, double *eprev,
                         double *state, double w0, double wmin, double wmax, double *U, hipStream_t s);
hipError_t launch_start_columns(double *U, const double *src, int64_t src_stride, int64_t src_off,
                                int64_t dst_stride, int T1, int64_t count, int replicate, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s);
size_t frac_lds_bytes(int fp32);
hipError_t launch_eval(const double *cu, const double *cv, int dim, int P, int T1, double t_prev, double h,
                       const double *pts, int64_t npts, double *out, hipStream_t s);
// batch_prefix: [n_groups + 3]; batch_split > 0 lets a round that fits in at
// most split_max items of batch_split paths use that batch (the 5-D
// matrix-core kernel then splits each item's products over the block's waves);
// share_max > 0: a round of few batches is split into shares of steps while
// batches times shares stay within share_max (share_done: its batch counters) and
// batches times rows times paths of a batch within share_cap, at most max_shares
constexpr int kMaxShares = 16;
// steps of a path sum's windows (divisors of 4, as rounds are multiples of 4).  Longer ones
// are fewer sums to store and add: a step each took 0.89 of the speed of unordered sums in
// the plane solve, four 0.97; in five dimensions, with rounds of 16 steps of 10^5 products,
// four leave too few to share out (138 -> 183 ms)
constexpr int window_steps(int dim) { return dim >= 4 ? 1 : 4; }
hipError_t launch_round_prep(const GroupDesc *groups, int32_t n_groups, int32_t round, int32_t steps,
                             int64_t mcount, int32_t batch, int32_t batch_split, int64_t split_max, int64_t share_max,
                             int64_t share_cap, int32_t rows, int32_t max_shares, const uint32_t *live_in, uint32_t *live_out, int64_t *batch_prefix, uint32_t *share_done,
                             unsigned long long *work, hipStream_t s);
// kern: 0 the vector-unit kernel, 1 the 2-D matrix-core kernel, 2 the 5-D one,
// 3 the windowed 1-D kernel
hipError_t launch_advance(const RoundArgs &a, int fp32, int samples_per_lane, int waves_per_block, int blocks,
                          size_t lds_bytes, int kern, hipStream_t s);
// windowed 1-D round kernel: residual form, centre-point rule, P <= 36, 1, 2 or
// 4 paths per lane; LDS: two windows of slabs
bool advance_1d_eligible(int dim, int P, int picard, int ball, int frac, int samples_per_lane);
size_t advance_1d_lds_bytes(int fp32, int64_t slab_stride);
// lattice form of the 1-D rounds (RoundArgs over nodes instead of groups)
int lat_window(int W);
hipError_t launch_lat_table(const RoundArgs &a, const LatArgs &la, hipStream_t s);
hipError_t launch_lat_advance(const RoundArgs &a, const LatArgs &la, int ns, int waves, int blocks, hipStream_t s);
// matrix-core form of the round kernel: FP32, d = 2, P <= 32, whole slab per
// LDS buffer, one path per lane
bool advance_mma_eligible(int fp32, int dim, int P, int cf, int samples_per_lane, int waves_per_block);
size_t advance_mma_lds_bytes(int P, int split);
// matrix-core slab layout (d = 2), the kernel's LDS image of one step, coefficients of
// T_{k0} T_{k1}.  P >= 17: halves [table u, v][part 0, 1][block of 8 modes
// k1][row k0 < 32][8 modes], the two parts a0 + a1 of the scaled coefficients;
// smaller P: FP32 columns (u modes k1, then v modes k1) of 33 rows k0.  Zeros past P.
// The line: against 64 bits the split products' rms error is 0.87-0.97 (random tables) and
// 0.82-0.97 (smooth ones) of the FP32 products' at P = 17 .. 32; at P = 5 and 10, split from
// FP32 values and summed in one chain, it was 1.1-1.15 times theirs, and the products
// are not what bounds a step there.
constexpr int kMmaRows = 33;
constexpr int kMmaSplitKH = 9;   // from this ceil(P / 2) on
constexpr bool mma_split(int P) { return (P + 1) / 2 >= kMmaSplitKH; }
constexpr int mma_blocks(int P) { return (P + 7) / 8; }
constexpr int64_t mma_slab_elems(int P, bool split)   // in floats
{
    return split ? (int64_t)512 * mma_blocks(P) : (int64_t)2 * ((P + 3) / 4 * 4) * kMmaRows;
}
// largest exponent e of |scaled coefficient| < 2^e
constexpr int kMmaScaleExp = 14;

// Five-dimensional matrix-core slab layout.  A step's image is a sequence of
// NCH chunks, each a 32-row tile of the two coefficient tables in two half-precision
// parts, [table u, v][part 0, 1][block of 8 modes][row < 32][8 modes] of halves,
// scaled as in the 2-D image.  Tile rows run over (k0, k1, k2), the modes over
// (k3, k4), k3 P + k4.  The rows f = k1 P + k2 < 32 A of each k0 fill A main tiles
// per k0, k0-major; the B = P^2 - 32 A remaining rows of every k0 are gathered,
// k0-major, into R tiles at the end, so every P in 3..12 wastes at most 3% of the
// rows.  Entries past P^2 modes and past the last row are zero.  P = 3 (27 products a
// path and table, and few modes to round) keeps FP32 entries, [table u, v][mode][row <
// 32]: the parts were up to 2.6 times as far from 64 bits there as FP32 products.
constexpr bool mma5_split(int P) { return P >= 4; }
struct Mma5Geom {
    int P, NB, A, B, R, NCH;
    int64_t table;   // floats of a chunk's u or v
    int64_t chunk;   // floats per chunk
    int64_t step;    // floats per step
};
constexpr Mma5Geom mma5_geom(int P)
{
    const int NB = (P * P + 7) / 8;
    const int A = P * P / 32, B = P * P - 32 * A, R = (B * P + 31) / 32;
    const int64_t table = mma5_split(P) ? (int64_t)256 * NB : (int64_t)32 * ((P * P + 1) / 2 * 2);
    return Mma5Geom{P, NB, A, B, R, P * A + R, table, 2 * table, (P * A + R) * 2 * table};
}
// Entry e of a step (one coefficient, [chunk][table][block][row][mode of the block] or
// [chunk][table][mode][row]): false for padding, else its table (0 u, 1 v), the flat index
// row4 = ((k0 P + k1) P + k2) P + k3 of the first four modes, and k4.
__host__ __device__ inline bool mma5_source(const Mma5Geom &g, int64_t e, int &uv, int64_t &row4, int &k4)
{
    const int c = (int)(e / g.chunk);
    int r = (int)(e - (int64_t)c * g.chunk);
    uv = r / (int)g.table;
    r -= uv * (int)g.table;
    const bool parts = mma5_split(g.P);
    const int i = parts ? (r >> 3) & 31 : r & 31, mode = parts ? 8 * (r >> 8) + (r & 7) : r >> 5;
    if (mode >= g.P * g.P) return false;
    const int k3 = mode / g.P;
    k4 = mode - k3 * g.P;
    int k0, f;
    if (c < g.P * g.A) {
        k0 = c / g.A;
        f = 32 * (c - k0 * g.A) + i;
    } else {
        const int rr = 32 * (c - g.P * g.A) + i;
        if (rr >= g.B * g.P) return false;
        k0 = rr / g.B;
        f = 32 * g.A + (rr - k0 * g.B);
    }
    row4 = ((int64_t)k0 * g.P * g.P + f) * g.P + k3;
    return true;
}
// matrix-core form of the 5-D round kernel: FP32, 3 <= P <= 12, residual form
// with the centre-point rule, one path per lane
bool advance_mma5_eligible(int fp32, int dim, int P, int picard, int ball, int samples_per_lane, int waves_per_block);
size_t advance_mma5_lds_bytes(int P);
hipError_t launch_slice_reduce(const double *result, int64_t n_nodes, int64_t mcount, double *sums, int first,
                               hipStream_t s);
size_t path_state_bytes(int fp32, int dim);
hipError_t launch_adjoint(const AdjointArgs &a, int fp32, int waves_per_block, int blocks, size_t lds_bytes,
                          hipStream_t s);
size_t adjoint_lds_bytes(int fp32, int mfma, int dim, int P, int nthr, int64_t slab_stride);
size_t adjoint_mma2_lds_bytes(int P, int nthr);
// the 2-D adjoint with u* on the matrix cores covers KH = ceil(P/2) <= 10 (past
// that its registers spill; larger P keep u* on the vector units)
constexpr int kAdjMma2MaxKH = 10;
hipError_t launch_slab_adjoint(const SlabArgs &a, int32_t groups_per_inst, int32_t n_inst, int fp32, double *cbar_u,
                               double *cbar_v, int64_t coef_inst_stride, int32_t shares, double *part, hipStream_t s);
int slab_adjoint_shares(const SlabArgs &a, int32_t groups_per_inst, int32_t n_inst, int max_nstar, int cus);
hipError_t launch_loss_lambda(const double *U, const double *target, int n_inst, int64_t nsp, int T1, double *lambda,
                              double *loss, hipStream_t s);
hipError_t launch_column_sum(const double *lambda, int64_t rows, int T1, double *out, hipStream_t s);
hipError_t launch_axpy(double *y, const double *x, int64_t n, hipStream_t s);

}  // namespace hpsmc
