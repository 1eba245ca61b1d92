// Matrix-core form of the 5-D FP32 round kernel (v_mfma_f32_32x32x16_f16 on split factors;
// v_mfma_f32_32x32x2f32 at P = 3).
#include "hpsmc_device.h"

namespace hpsmc {

// ===========================================================================
// The residual of a walk step needs u and v at the path's point X, each a
// contraction of the step's slab S[k0..k4] with the tensor product of the
// Legendre values L_{k_i}(X_i) (eq. interIQ, the tensor-product basis of the
// discrete space).  Over the 64 paths of a wave the innermost two modes form
// a dense product: with B[(k3,k4)][s] = L_{k3}(X3_s) L_{k4}(X4_s),
//     T[(k0,k1,k2)][s] = sum_{k3,k4} S[k0,k1,k2,k3,k4] B[(k3,k4)][s],
// a (rows x P^2)(P^2 x 64) product, then per path
//     u_s = sum_{k0,k1,k2} L_{k0} L_{k1} L_{k2} T[(k0,k1,k2)][s],
// P^3 multiply-adds on the vector unit.  The product takes 4 P^5 of the 4 P^5
// + O(P^3) operations of a residual evaluation; it runs on the matrix cores in
// 32-row tiles (the slab layout of mma5_geom) streamed through LDS.
//
// From P = 4 on both factors are split into two half-precision parts (as in the 2-D
// kernel, whose operand layout it shares): a product of 32x32x16 takes eight modes, lanes 0-31
// feeding part 0 of the B entries and lanes 32-63 part 1 against the same part of
// the slab.  Paths 0-31 form product "A", paths 32-63 product "B".  The B entries are
// formed and split once per step and stay in registers for all tiles: at P = 10, 50
// split pairs and swaps a step and 104 products of 32x32x16 a tile, where FP32
// products (32x32x2) took 200 a tile, of twice the time each, and formed every entry
// again for every tile: 8^5 x 8 nodes, two samples, 302 -> 155 ms an iteration.  Error
// against 64 bits (rms, of the FP32 products', random and smooth tables): 0.6 and 0.5 at
// P = 4, 0.8 and 0.5 at 5, 0.75-0.8 at 6 and 7, 1.0 and 0.9 at 8, 0.75 and 0.65 at 10.
// ===========================================================================
template <int P>
__device__ __forceinline__ void legendre_row(float x, float (&L)[P])
{
    L[0] = 1.f;
    if (P > 1) L[1] = x;
#pragma unroll
    for (int k = 1; k + 1 < P; ++k)
        L[k + 1] = (float)((2.0 * k + 1.0) / (k + 1.0)) * x * L[k] - (float)(k / (k + 1.0)) * L[k - 1];
}

// B operands: entries L_{k3}(x3) L_{k4}(x4) of the wave's 64 points, modes k3 P + k4 in
// pairs: scaled by bscale, in two parts; or in FP32, lanes 0-31 the even mode of a pair,
// lanes 32-63 the odd one
template <int P> struct Mma5B {
    static constexpr bool SPLIT = mma5_split(P);
    static constexpr int NB = mma5_geom(P).NB, NR = SPLIT ? 4 * NB : (P * P + 1) / 2;
    uint32_t r[NR];
    __device__ __forceinline__ h16x8 block(int b) const
    {
        const u32x4 q = {r[4 * b], r[4 * b + 1], r[4 * b + 2], r[4 * b + 3]};
        return __builtin_bit_cast(h16x8, q);
    }
};
template <int P>
__device__ __forceinline__ void mma5_operands(float x3, float x4, float bscale, Mma5B<P> &bA, Mma5B<P> &bB)
{
    float L3[P], L4[P];
    legendre_row<P>(x3, L3);
    legendre_row<P>(x4, L4);
    if constexpr (Mma5B<P>::SPLIT) {
#pragma unroll
        for (int k = 0; k < P; ++k) L3[k] *= bscale;   // a power of two
    }
    const float m1 = opaque_minus_one();
#pragma unroll
    for (int i = 0; i < Mma5B<P>::NR; ++i) {
        bA.r[i] = 0u;
        bB.r[i] = 0u;
        if (2 * i < P * P) {
            const int m0 = 2 * i, n0 = 2 * i + 1 < P * P ? 2 * i + 1 : 2 * i;
            const float e0 = L3[m0 / P] * L4[m0 % P], e1 = n0 > m0 ? L3[n0 / P] * L4[n0 % P] : 0.f;
            uint32_t h = __float_as_uint(e0), l = __float_as_uint(e1);
            if constexpr (Mma5B<P>::SPLIT) {
                h = pack_h16(e0, e1);
                l = pack_h16_rest(e0, e1, h, m1);
            }
            const auto r = __builtin_amdgcn_permlane32_swap(h, l, false, false);
            bA.r[i] = r[0];
            bB.r[i] = r[1];
        }
    }
}

// the products of one tile and table with both path halves (S: the tile's two parts),
// over the blocks b of part `part` of `nparts` (b % nparts == part: the waves that
// share one item in a sparse round); the small part of the slab first.  Slab operands
// are read two blocks ahead of their products; the fence keeps the scheduler from
// hoisting all of a tile's reads.
template <int P, bool PARTS>
__device__ __forceinline__ void mma5_tile(const u32x4 *S, int lane, const Mma5B<P> &bA, const Mma5B<P> &bB, int part,
                                          int nparts, f32x16 &dA, f32x16 &dB)
{
    constexpr int NB = mma5_geom(P).NB, N = 2 * NB;
    dA = f32x16{};
    dB = f32x16{};
    if constexpr (!Mma5B<P>::SPLIT) {   // FP32 products of a pair of modes each
        const float *A = (const float *)S + lane;   // mode 2 i + lane / 32, row lane % 32
#pragma unroll
        for (int i = 0; i < Mma5B<P>::NR; ++i) {
            if (!PARTS || i % nparts == part) {
                dA = __builtin_amdgcn_mfma_f32_32x32x2f32(A[64 * i], __uint_as_float(bA.r[i]), dA, 0, 0, 0);
                dB = __builtin_amdgcn_mfma_f32_32x32x2f32(A[64 * i], __uint_as_float(bB.r[i]), dB, 0, 0, 0);
            }
        }
        return;
    }
    const u32x4 *A = S + (lane & 31);
    // operand n: block n % NB of part 1 (n < NB), then of part 0
    auto addr = [](int n) { return ((n < NB ? NB : 0) + n % NB) * 32; };
    u32x4 x[2];
    x[0] = A[addr(0)];
    if (N > 1) x[1] = A[addr(1)];
#pragma unroll
    for (int n = 0; n < N; ++n) {
        const int b = n % NB;
        const h16x8 a8 = __builtin_bit_cast(h16x8, x[n & 1]);
        if (!PARTS || b % nparts == part) {
            dA = __builtin_amdgcn_mfma_f32_32x32x16_f16(a8, bA.block(b), dA, 0, 0, 0);
            dB = __builtin_amdgcn_mfma_f32_32x32x16_f16(a8, bB.block(b), dB, 0, 0, 0);
        }
        if (n + 2 < N) x[n & 1] = A[addr(n + 2)];
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Rows of a tile back to the lane that owns the path: register r holds rows
// 8(r/4) + r%4 (from the lane's own half) and 8(r/4) + 4 + r%4 (from the other
// half) of the path's column after one swap of the A and B products.
// Main tile t of a k0: rows f = 32 t + i = (k1, k2); au[k1] += L_{k2} T.
template <int P>
__device__ __forceinline__ void mma5_fold_main(int t, const f32x16 &dA, const f32x16 &dB, const float (&L2)[P],
                                               float (&acc)[P])
{
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int ia = 8 * (r >> 2) + (r & 3), ib = ia + 4;
        const int fa = 32 * t + ia, fb = 32 * t + ib;
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(dA[r]), __float_as_uint(dB[r]), false, false);
        acc[fa / P] = fmaf(L2[fa % P], __uint_as_float(p[0]), acc[fa / P]);
        acc[fb / P] = fmaf(L2[fb % P], __uint_as_float(p[1]), acc[fb / P]);
    }
}

// Remainder tile t: rows rr = 32 t + i hold (k0, f) = (rr / B, 32 A + rr % B),
// weight L_{k0} L_{k1} L_{k2}; rows past B P are zero and skipped.  Four sums (the two
// halves of the swap, the first tile and the others): chains of up to 125 terms into
// one would round each of them.
template <int P>
__device__ __forceinline__ void mma5_fold_rem(int t, const f32x16 &dA, const f32x16 &dB, const float (&L0)[P],
                                              const float (&L1)[P], const float (&L2)[P], float (&u)[4])
{
    constexpr Mma5Geom g = mma5_geom(P);
    const int s = t > 0 ? 2 : 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int ia = 8 * (r >> 2) + (r & 3), ib = ia + 4;
        const int ra = 32 * t + ia, rb = 32 * t + ib;
        if (ra >= g.B * P) continue;   // rb > ra
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(dA[r]), __float_as_uint(dB[r]), false, false);
        {
            const int k0 = ra / g.B, f = 32 * g.A + ra % g.B;
            u[s] = fmaf(L0[k0] * (L1[f / P] * L2[f % P]), __uint_as_float(p[0]), u[s]);
        }
        if (rb < g.B * P) {
            const int k0 = rb / g.B, f = 32 * g.A + rb % g.B;
            u[s + 1] = fmaf(L0[k0] * (L1[f / P] * L2[f % P]), __uint_as_float(p[1]), u[s + 1]);
        }
    }
}

// ===========================================================================
// Round kernel, matrix-core form: d = 5, FP32, residual form with the
// centre-point rule, one path per lane.  The walk (directions from two
// Philox blocks per step, jump, exit test of eq. indexL, left-point
// quadrature of eq. interIQ, path sums in FP64) is the vector-unit
// kernel's, so both take the same exit steps and differ in u, v only by
// rounding.  A step's NCH chunks stream through two LDS buffers
// along one sequence that runs on into the next step: while a chunk's
// products run, the next chunk is in flight (global_load_lds), and one
// barrier per chunk publishes it.
// ===========================================================================
template <int P>
__device__ __forceinline__ void advance_mma5_body(const RoundArgs &a)
{
    constexpr Mma5Geom g5 = mma5_geom(P);
    constexpr int A = g5.A, R = g5.R, NCH = g5.NCH, TV = (int)g5.table / 4;   // TV: 16-byte vectors of a tile's table
    constexpr int CF = (int)g5.chunk, CV = CF / 4;   // floats, 16-byte vectors per chunk
    extern __shared__ u32x4 lds[];
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6;
    __shared__ long long s_item;
    __shared__ SrcTime<float> s_tf[256];   // source time factors of a window of blockDim.x steps
    __shared__ double s_acc[256];          // path sums
    __shared__ uint16_t s_len[256];        // shares: the steps each path takes in the round
    __shared__ float s_red[2][4][64];      // sparse rounds: each wave's share of u and v
    cptr<GroupDesc> groups = as_const(a.groups);
    cptr<NodeDesc> nodes = as_const(a.nodes);
    const int64_t total = a.batch_prefix[a.n_groups];
    const int shares = (int)a.batch_prefix[a.n_groups + 2];
    // Sparse rounds (few live paths, set by the round's prep kernel): an item is
    // 64 paths that every wave of the block walks alike; wave w runs its share
    // of each tile's k-steps, the shares are summed in wave order, and wave 0
    // alone writes results, state and counts.
    const int bsz = (int)a.batch_prefix[a.n_groups + 1];
    const bool split = bsz < nthr;
    const int nparts = split ? nthr >> 6 : 1, part = split ? wave : 0;
    const bool writer = !split || wave == 0;
    unsigned long long evals = 0, slots = 0;
    using State = PathState<float, 5>;
    const State *sin = (const State *)a.state_in;
    State *sout = (State *)a.state_out;

    for (bool first = true;; first = false) {
        const int64_t item = take_item(a, total, first, s_item);
        if (item >= total) break;
        const int64_t batch = item / shares;
        const int share = (int)(item - batch * shares);
        int lo = 0, hi = a.n_groups - 1;   // last g with batch_prefix[g] <= batch
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.batch_prefix[mid] <= batch) lo = mid; else hi = mid - 1;
        }
        const int g = lo;
        const int64_t b = batch - a.batch_prefix[g];
        cptr<GroupDesc> G = groups + g;
        const int nstar = G->nstar;
        const int q0 = a.round * a.steps;
        const int q1 = min(q0 + a.steps, nstar);
        const float delta = (float)G->delta, J = (float)G->jump;
        const double span = G->span, t_prev = G->t_prev, ddelta = G->delta;
        const uint32_t c3 = G->c3 | (uint32_t)a.tag;
        const int64_t live = a.round == 0 ? (int64_t)G->node_count * a.mcount : (int64_t)a.live_in[g];
        const float *gtab = (const float *)a.slab_table + G->slab_mma;
        float iu = 1.f, iv = 1.f;
        if constexpr (Mma5B<P>::SPLIT) {
            iu = a.inv_scale[2 * G->blk];
            iv = a.inv_scale[2 * G->blk + 1];
        }

        // ---- this lane's path
        const int64_t p = b * bsz + (split ? lane : tid);
        const bool began = p < live;
        bool alive = began;
        uint32_t node = 0, sample = 0, c0 = 0;
        float X[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
        using Sums = PathSums<1, window_steps(5)>;
        Sums ps;
        ps.start(s_acc, a, batch, bsz, split ? lane : tid, nthr);
        if (alive) {
            if (a.round == 0) {
                node = (uint32_t)(G->node_begin + p / a.mcount);
                sample = (uint32_t)(a.m0 + p % a.mcount);
#pragma unroll
                for (int i = 0; i < 5; ++i) X[i] = (float)nodes[node].x0[i];
            } else {
                const State st = sin[G->path_off + p];
#pragma unroll
                for (int i = 0; i < 5; ++i) X[i] = st.x[i];
                ps.acc(0) = st.sum();
                node = st.node;
                sample = st.sample;
            }
            c0 = nodes[node].c0;
        }
        if (shares > 1) s_len[tid] = (uint16_t)(alive ? q1 - q0 : 0);
        auto fill_time = [&](int qs) {
            const int qq = qs + tid;
            if (qq < q1) s_tf[tid] = source_time<float>(a.phys, (float)(t_prev + (span - (double)qq * ddelta)));
        };
        fill_time(q0);
        // chunk 0 of the first evaluated step into buffer 0; buf: the buffer of the current chunk
        int qe = q0 + share * window_steps(5);   // the next step this share evaluates
        if (qe < q1) mma_stage((const u32x4 *)(gtab + (int64_t)qe * a.slab_stride), lds, CV, tid, nthr);
        mma_stage_wait();
        __syncthreads();
        int buf = 0;

        int q = q0, tslot = 0;
        for (; q < q1; ++q, ++tslot) {
            if (tslot == nthr) {   // the previous step's barrier ended every read of the old window
                tslot = 0;
                fill_time(q);
                __syncthreads();
            }
            // ---- direction (Philox blocks 2q, 2q + 1), jump and exit test (eq. indexL)
            float Y[5];
            if (alive) {
                float dir[5];
                sphere_dir<float, 5>(c0, sample, q, c3, a.key0, a.key1, dir);
                bool inside = true;
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    Y[i] = m_fma(J, dir[i], X[i]);
                    inside = inside && (fabsf(Y[i]) < 1.f);
                }
                alive = inside;   // else the path ended: L = q
                if (shares > 1 && !inside) s_len[tid] = (uint16_t)(q - q0);
            }
            if (writer && share == 0) ++slots;
            if (q != qe) {   // another share's step: the walk alone
                if (alive) {
#pragma unroll
                    for (int i = 0; i < 5; ++i) X[i] = Y[i];
                }
                continue;
            }
            qe = q0 + Sums::next(q - q0, shares);
            // ---- u and v at X_q: the step's chunks, the next one always in flight
            const bool wave_live = __ballot(alive) != 0ull;
            Mma5B<P> bA, bB;
            float L1[P], L2[P];
            mma5_operands<P>(X[3], X[4], a.bscale, bA, bB);
            legendre_row<P>(X[1], L1);
            legendre_row<P>(X[2], L2);
            const float *step_src = gtab + (int64_t)q * a.slab_stride;
            const bool more = qe < q1;
            auto stage_next = [&](int c) {   // chunk c + 1 of this step, or chunk 0 of the next evaluated one
                const float *src = c + 1 < NCH ? step_src + (int64_t)(c + 1) * CF
                                               : (more ? gtab + (int64_t)qe * a.slab_stride : nullptr);
                if (src) mma_stage((const u32x4 *)src, lds + (buf ^ 1) * CV, CV, tid, nthr);
            };
            auto tile = [&](const u32x4 *S, const Mma5B<P> &pA, const Mma5B<P> &pB, f32x16 &dA, f32x16 &dB) {
                if (nparts == 1) mma5_tile<P, false>(S, lane, pA, pB, 0, 1, dA, dB);
                else mma5_tile<P, true>(S, lane, pA, pB, part, nparts, dA, dB);
            };
            float us[4] = {}, vs[4] = {};   // sums of rising modes, added up from the last
            if constexpr (A > 0) {
                float l0p = 0.f, l0c = 1.f;   // L_{k0}(X0)
                for (int k0 = 0; k0 < P; ++k0) {
                    float au[P], av[P];
#pragma unroll
                    for (int k = 0; k < P; ++k) { au[k] = 0.f; av[k] = 0.f; }
#pragma unroll
                    for (int t = 0; t < A; ++t) {
                        stage_next(k0 * A + t);
                        if (wave_live) {
                            f32x16 dA, dB;
                            tile(lds + buf * CV, bA, bB, dA, dB);
                            mma5_fold_main<P>(t, dA, dB, L2, au);
                            tile(lds + buf * CV + TV, bA, bB, dA, dB);
                            mma5_fold_main<P>(t, dA, dB, L2, av);
                        }
                        mma_stage_wait();
                        __syncthreads();
                        buf ^= 1;
                    }
                    float su = 0.f, sv = 0.f;
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        su = fmaf(L1[k], au[k], su);
                        sv = fmaf(L1[k], av[k], sv);
                    }
                    if (k0 < 2) {
                        us[0] = fmaf(l0c, su, us[0]);
                        vs[0] = fmaf(l0c, sv, vs[0]);
                    } else {
                        us[1] = fmaf(l0c, su, us[1]);
                        vs[1] = fmaf(l0c, sv, vs[1]);
                    }
                    const float nx = (float)((2.0 * k0 + 1.0) / (k0 + 1.0)) * X[0] * l0c - (float)(k0 / (k0 + 1.0)) * l0p;
                    l0p = l0c;
                    l0c = nx;
                }
            }
            if constexpr (R > 0) {
                float L0[P], ur[4] = {}, vr[4] = {};
                legendre_row<P>(X[0], L0);
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    stage_next(P * A + t);
                    if (wave_live) {
                        f32x16 dA, dB;
                        tile(lds + buf * CV, bA, bB, dA, dB);
                        mma5_fold_rem<P>(t, dA, dB, L0, L1, L2, ur);
                        tile(lds + buf * CV + TV, bA, bB, dA, dB);
                        mma5_fold_rem<P>(t, dA, dB, L0, L1, L2, vr);
                    }
                    mma_stage_wait();
                    __syncthreads();
                    buf ^= 1;
                }
                us[2] = ur[0] + ur[2];
                us[3] = ur[1] + ur[3];
                vs[2] = vr[0] + vr[2];
                vs[3] = vr[1] + vr[3];
            }
            float u = us[0] + (us[1] + (us[2] + us[3])), v = vs[0] + (vs[1] + (vs[2] + vs[3]));
            if (split) {   // the waves' shares of u and v, summed in wave order
                s_red[0][wave][lane] = u;
                s_red[1][wave][lane] = v;
                __syncthreads();
                u = 0.f;
                v = 0.f;
                for (int k = 0; k < nparts; ++k) {
                    u += s_red[0][k][lane];
                    v += s_red[1][k][lane];
                }
            }
            u *= iu;
            v *= iv;
            if (alive) {   // residual at X_q, time tau_q = t_{n,l} - q Delta
                const float r = f_of<float>(a.phys, u) + source_space<float, 5>(a.phys, X, s_tf[tslot]) + v;
                if (writer) ps.add(0, (double)delta, (double)r);
#pragma unroll
                for (int i = 0; i < 5; ++i) X[i] = Y[i];
                if (writer) ++evals;
            }
            if (Sums::last(q - q0) || q + 1 == q1) ps.close(q - q0, shares);
            if (__syncthreads_or(alive ? 1 : 0) == 0) {
                ps.close(q - q0, shares);
                ++q;
                break;
            }
        }

        // ---- paths ended in this round or at N*, and those carried to the next round
        if (shares > 1) {
            if (!share_last(a, batch, shares, s_item)) continue;
            const int len[1] = {writer ? s_len[tid] : 0};
            share_fold(ps, len);
        }
        const bool carry = writer && alive && q1 < nstar;
        if (writer && began && !carry) a.result[(int64_t)nodes[node].out * a.mcount + (sample - a.m0)] = ps.acc(0);
        const unsigned long long mask = __ballot(carry);
        if (mask != 0ull) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(a.live_out + g, (uint32_t)__popcll(mask));
            base = __shfl(base, 0, 64);
            if (carry) {
                const uint32_t off = base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                State st;
#pragma unroll
                for (int i = 0; i < 5; ++i) st.x[i] = X[i];
                st.put_sum(ps.acc(0));
                st.node = node;
                st.sample = sample;
                sout[G->path_off + off] = st;
            }
        }
    }
    add_stats(a, evals, slots);
}

template <int P>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) advance_mma5_kernel(RoundArgs a)
{
    advance_mma5_body<P>(a);
}

bool advance_mma5_eligible(int fp32, int dim, int P, int picard, int ball, int samples_per_lane, int waves_per_block)
{
    return fp32 && dim == 5 && P >= 3 && P <= 12 && !picard && !ball && samples_per_lane == 1 &&
           waves_per_block >= 1 && waves_per_block <= 4;
}

size_t advance_mma5_lds_bytes(int P) { return (size_t)2 * mma5_geom(P).chunk * sizeof(float); }

template <int P>
static hipError_t adv_mma5(const RoundArgs &a, dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    if constexpr (P > 12) {
        return hipErrorInvalidValue;
    } else {
        if (a.P != P) return adv_mma5<P + 1>(a, grid, block, lds, s);
        if (lds < advance_mma5_lds_bytes(P) || a.slab_stride != mma5_geom(P).step) return hipErrorInvalidValue;
        hipLaunchKernelGGL((advance_mma5_kernel<P>), grid, block, lds, s, a);
        return hipGetLastError();
    }
}

hipError_t launch_adv_mma5(const RoundArgs &a, dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    if (a.phys.dim != 5 || a.phys.picard || a.phys.ball || a.P < 3 || block.x > 256 || block.x % 64 != 0)
        return hipErrorInvalidValue;
    return adv_mma5<3>(a, grid, block, lds, s);
}

}  // namespace hpsmc
