// One-dimensional round kernels on the walk's lattice (FP64): the residual
// form with the centre-point rule, tabulated instead of evaluated path by path.
#include "hpsmc_device.h"

namespace hpsmc {

// ===========================================================================
// On a line every jump is +-J, so the paths of one node visit only the points
// x_j + m J inside (-1, 1), of which step q reaches those with m = q (mod 2):
// about 1/J of them, while thousands of paths of the node are alive.  Instead of
// evaluating Delta r(X_q, tau_q) (eq. interIQ) once per path and step, a round
// first tabulates it at every lattice point of every node and step of the round
// (lat_table_kernel), and a path step (lat_advance_kernel) draws its bit, moves,
// tests the exit (eq. indexL) and adds one table entry: the same Philox words,
// the same positions X_{q+1} = X_q +- J and the same exits as the general
// kernel; the residual is taken at x_j + m J itself rather than at the position's
// accumulated sum (they differ by its rounding, about 1e-15).
// The table is bound by FP64 fma's (2 P per entry: a thread keeps the basis
// values of its point and runs over the steps, whose coefficients are scalar
// operands), the walk by its own ten-odd instructions and one LDS gather (eight
// steps' gathers in flight together).  16 x 16 nodes, 4096 samples, five
// iterations: 90 ms with every path evaluated, 14.5 ms so (tables 4, walk 9.7);
// a coarse iteration of 64 samples, 200 steps one after another: 667 -> 195 us.
// ===========================================================================

constexpr int kLatChunk = 64;   // steps a table block takes, half of them (one parity) evaluated

// One thread per entry of a step, the entries of a group's nodes in a row (full
// waves whatever the width of one node), blockIdx.x a chunk of steps and the
// parity of the steps it takes: a thread's point is then the same at every step.
template <int PM>
__global__ void __launch_bounds__(256) lat_table_kernel(RoundArgs a, LatArgs la)
{
    const int tid = threadIdx.x;
    cptr<GroupDesc> G = as_const(la.groups) + blockIdx.z;
    const int q0 = a.round * a.steps, nstar = G->nstar, node0 = G->node_begin, nn = G->node_count;
    const int qa = q0 + (int)(blockIdx.x >> 1) * kLatChunk, qb = min(min(qa + kLatChunk, q0 + a.steps), nstar);
    if (qa >= qb) return;
    const int64_t t0 = la.desc[node0].toff;
    const int e = blockIdx.y * 256 + tid;   // entry of the group's steps
    int lo = 0, hi = nn - 1;                // last node whose entries start at or before e
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (la.desc[node0 + mid].toff - t0 <= e) lo = mid; else hi = mid - 1;
    }
    const LatDesc d = la.desc[node0 + lo];
    const int i = e - (int)(d.toff - t0);
    const bool live = i < d.W && (a.round == 0 || a.live_in[node0 + lo] != 0u);
    if (__syncthreads_or(live ? 1 : 0) == 0) return;
    const double J = G->jump, delta = G->delta, span = G->span, t_prev = G->t_prev;
    __shared__ SrcTime<double> s_tf[kLatChunk];
    if (tid < qb - qa) s_tf[tid] = source_time<double>(a.phys, t_prev + (span - (double)(qa + tid) * delta));
    __syncthreads();
    const int first = qa + ((qa ^ (int)blockIdx.x) & 1);
    const double x[1] = {fma((double)(d.mlo + 2 * i + ((first - d.mlo) & 1)), J, a.nodes[node0 + lo].x0[0])};
    double Tk[PM];
    Tk[0] = 1.0;
    Tk[1] = x[0];
#pragma unroll
    for (int k = 2; k < PM; ++k) Tk[k] = fma(x[0] + x[0], Tk[k - 1], -Tk[k - 2]);
    const double *gtab = (const double *)a.slab_table + G->slab;
    double *tab = la.table + d.toff * a.steps + i;
    for (int q = first; q < qb; q += 2) {
        cptr<double> S = as_const(gtab + (int64_t)q * a.slab_stride);
        double u = 0.0, v = 0.0, u1 = 0.0, v1 = 0.0;
#pragma unroll
        for (int kb = 0; kb < PM / 2; ++kb) {
            if (kb * 2 < a.P) {   // rows are padded with zeros to a multiple of 4 modes
                u = fma(S[2 * kb], Tk[2 * kb], u);
                v = fma(S[a.PP + 2 * kb], Tk[2 * kb], v);
                u1 = fma(S[2 * kb + 1], Tk[2 * kb + 1], u1);
                v1 = fma(S[a.PP + 2 * kb + 1], Tk[2 * kb + 1], v1);
            }
        }
        const double r = f_of<double>(a.phys, u + u1) + source_space<double, 1>(a.phys, x, s_tf[q - qa]) + (v + v1);
        if (live) tab[(int64_t)(q - q0) * d.W] = delta * r;
    }
}

template <int NS>
__global__ void __launch_bounds__(256) lat_advance_kernel(RoundArgs a, LatArgs la)
{
    extern __shared__ u32x4 lds[];
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    __shared__ long long s_item;
    cptr<GroupDesc> groups = as_const(a.groups);
    cptr<NodeDesc> nodes = as_const(a.nodes);
    const int64_t total = a.batch_prefix[a.n_groups];
    unsigned long long evals = 0, slots = 0;
    using State = PathState<double, 1>;
    const State *sin = (const State *)a.state_in;
    State *sout = (State *)a.state_out;
    double *zero = (double *)lds + 2 * la.win * la.wmax;   // what ended paths add
    if (tid == 0) *zero = 0.0;

    for (bool first = true;; first = false) {
        const int64_t item = take_item(a, total, first, s_item);
        if (item >= total) break;
        int lo = 0, hi = a.n_groups - 1;   // last node with batch_prefix <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.batch_prefix[mid] <= item) lo = mid; else hi = mid - 1;
        }
        const int g = __builtin_amdgcn_readfirstlane(lo);
        const int64_t b = item - a.batch_prefix[g];
        cptr<GroupDesc> G = groups + g;
        const int nstar = G->nstar;
        const int q0 = a.round * a.steps;
        const int q1 = min(q0 + a.steps, nstar);
        const double J = G->jump;
        const uint32_t c3 = G->c3 | (uint32_t)a.tag;
        const uint32_t node = (uint32_t)G->node_begin, c0 = nodes[node].c0;
        const double x0 = nodes[node].x0[0];
        const int64_t out = (int64_t)nodes[node].out * a.mcount;
        const int64_t live = a.round == 0 ? a.mcount : (int64_t)a.live_in[g];
        const int mlo = la.desc[g].mlo, W = la.desc[g].W;
        const double *tab = la.table + la.desc[g].toff * a.steps;
        const int wvec = la.win * W / 2;   // 16-byte vectors per window buffer (W is even)
        const int jhi = __double2hiint(J), jlo = __double2loint(J);

        double X[NS], acc[NS];
        int up[NS];   // jumps to the right so far: m = 2 up - q
        bool alive[NS], began[NS];
        uint32_t sample[NS], w[NS][4], bits[NS], cnt = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int64_t p = b * a.batch + (int64_t)s * nthr + tid;
            began[s] = alive[s] = p < live;
            X[s] = x0; acc[s] = 0.0; sample[s] = 0;
            if (alive[s]) {
                if (a.round == 0) {
                    sample[s] = (uint32_t)(a.m0 + p);
                } else {
                    const State st = sin[G->path_off + p];
                    X[s] = st.x[0];
                    acc[s] = st.acc;
                    sample[s] = st.sample;
                }
            }
            up[s] = ((int)rint((X[s] - x0) / J) + q0) >> 1;
        }
        // window [qw, qw + win) of the node's table rows, contiguous, into buffer wb
        auto stage = [&](int qw, int wb) {
            const int n = min(la.win, q1 - qw);
            mma_stage((const u32x4 *)(tab + (int64_t)(qw - q0) * W), lds + wb * wvec, n * W / 2, tid, nthr);
        };
        stage(q0, 0);
        mma_stage_wait();
        __syncthreads();

        int wb = 0;
#pragma unroll 1
        for (int qw = q0; qw < q1; qw += la.win, wb ^= 1) {
            const int n = min(la.win, q1 - qw);
            if (qw + la.win < q1) stage(qw + la.win, wb ^ 1);   // its last readers passed the previous barrier
            // directions: bit q % 32 of word (q / 32) % 4 of the Philox block q / 128; windows
            // do not cross a word (win divides 32, rounds are multiples of 32)
            if ((qw & 127) == 0 || qw == q0) {
#pragma unroll
                for (int s = 0; s < NS; ++s) philox(c0, sample[s], (uint32_t)(qw >> 7), c3, a.key0, a.key1, w[s]);
            }
            const int wi = (qw >> 5) & 3;
#pragma unroll
            for (int s = 0; s < NS; ++s)
                bits[s] = (wi == 0 ? w[s][0] : wi == 1 ? w[s][1] : wi == 2 ? w[s][2] : w[s][3]) >> (qw & 31);
            // entry of m - mlo = 2 up - q - mlo in the step's row: up + floor((-q - mlo) / 2)
            const double *S = (const double *)(lds + wb * wvec);
            auto group = [&](int k0, auto count) {   // steps k0 .. k0 + count - 1: gathers in flight together
                constexpr int N = decltype(count)::value;
                double y[N][NS];
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const int k = k0 + j;
                    const double *row = S + k * W + ((-(qw + k) - mlo) >> 1);
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        // X +- J: J with the bit's sign (fma(J, +-1, X) exactly)
                        X[s] += __hiloint2double(jhi ^ (int)(~(bits[s] << (31 - k)) & 0x80000000u), jlo);
                        alive[s] = alive[s] && fabs(X[s]) < 1.0;   // else the path ended: L = q
                        y[j][s] = *(alive[s] ? row + up[s] : zero);
                        up[s] += (int)(bits[s] >> k & 1u);
                        cnt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(alive[s]));
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < N; ++j) {
#pragma unroll
                    for (int s = 0; s < NS; ++s) acc[s] += y[j][s];
                }
            };
            constexpr int kG = NS == 1 ? 8 : 4;
            if (n == 16) {
#pragma unroll
                for (int k = 0; k < 16; k += kG) group(k, std::integral_constant<int, kG>{});
            } else {
#pragma unroll 1
                for (int k = 0; k < n; ++k) group(k, std::integral_constant<int, 1>{});
            }
            slots += (unsigned long long)(NS * n);
            bool any_live = false;
#pragma unroll
            for (int s = 0; s < NS; ++s) any_live = any_live || alive[s];
            mma_stage_wait();   // the next window has landed
            if (__syncthreads_or(any_live ? 1 : 0) == 0) break;
        }
        if (lane == 0) evals += cnt;   // counted per wave

        // ---- paths ended in this round or at N*, and those carried to the next round
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const bool carry = alive[s] && q1 < nstar;
            if (began[s] && !carry) a.result[out + (sample[s] - a.m0)] = acc[s];
            const unsigned long long mask = __ballot(carry);
            if (mask != 0ull) {
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(a.live_out + g, (uint32_t)__popcll(mask));
                base = __shfl(base, 0, 64);
                if (carry) {
                    const uint32_t off = base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                    State st;
                    st.x[0] = X[s];
                    st.acc = acc[s];
                    st.comp = 0.0;
                    st.node = node;
                    st.sample = sample[s];
                    sout[G->path_off + off] = st;
                }
            }
        }
    }
    add_stats(a, evals, slots);
}

// steps per LDS window: 16 where two buffers of the widest node's rows stay
// within 32 KiB (so that blocks share the CU), fewer for wider rows
int lat_window(int W)
{
    int win = 16;
    while (win > 1 && (int64_t)2 * win * W * 8 > 32 * 1024) win /= 2;
    return win;
}

hipError_t launch_lat_table(const RoundArgs &a, const LatArgs &la, hipStream_t s)
{
    const dim3 grid((unsigned)(2 * ((a.steps + kLatChunk - 1) / kLatChunk)), (unsigned)((la.emax + 255) / 256),
                    (unsigned)la.n_groups);
    if (a.P <= 12) hipLaunchKernelGGL(lat_table_kernel<12>, grid, dim3(256), 0, s, a, la);
    else if (a.P <= 20) hipLaunchKernelGGL(lat_table_kernel<20>, grid, dim3(256), 0, s, a, la);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_lat_advance(const RoundArgs &a, const LatArgs &la, int ns, int waves, int blocks, hipStream_t s)
{
    const dim3 grid(blocks), block(64 * waves);
    const size_t lds = (size_t)2 * la.win * la.wmax * 8 + 16;
    if (a.steps % 32 != 0 || a.batch != 64 * waves * ns || lds > 65536) return hipErrorInvalidValue;
    switch (ns) {
    case 1: hipLaunchKernelGGL(lat_advance_kernel<1>, grid, block, lds, s, a, la); break;
    case 2: hipLaunchKernelGGL(lat_advance_kernel<2>, grid, block, lds, s, a, la); break;
    case 4: hipLaunchKernelGGL(lat_advance_kernel<4>, grid, block, lds, s, a, la); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace hpsmc
