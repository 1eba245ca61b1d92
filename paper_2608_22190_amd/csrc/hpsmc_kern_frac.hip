// Fractional form of the round kernel (Ex. 2-3, d = 1).
#include "hpsmc_device.h"

namespace hpsmc {

// ===========================================================================
// Round kernel, fractional form (Ex. 2-3): d = 1, u_t = -(-Delta)^{alpha/2} u
// + f(u) + s, one path per lane.  The walk jumps by J = R / sqrt(x) with
// x = I^{-1}(omega; alpha/2, 1 - alpha/2) (the exit law of a ball of radius R
// for the alpha-stable process started at its centre; the mean exit time of
// that ball is Delta), in a fair direction.  The slab of a step holds the
// symmetric Jacobi coefficients (parameter a = alpha/2) of u*/w and of
// -d_t u*/w, w = (1 - x^2)^a, and the residual is
//   r = f(w U) + s + w V - sum_k lambda_k U_k P_k,  lambda_k = Gamma(k+alpha+1)/k!
// (the fractional Laplacian of the generalized Jacobi function w P_k).
// Philox: block q/2, words 2(q mod 2) (omega) and 2(q mod 2) + 1 (sign bit).
// ===========================================================================

// log x solving I_x(p, 1-p) = y for x <= 1/2.  With the series
// I_x = x^p (1-x)^{1-p} / (p B) sum_k t_k, t_{k+1} = t_k x (k+1)/(p+1+k), and the
// small-x asymptote z0 = (log y + log(p B)) / p, X0 = e^{z0}, the solution is
// x = X0 e^{-h(x)/p}, h(x) = (1-p) log(1-x) + log sum_k t_k, an analytic
// function of X0 on [0, X0max] (X0max the asymptote at x = 1/2): log(x / X0) comes
// from a cubic in each of kFracTab intervals, within 10^-11.  In FP32 that is below
// the rounding of z0, and the logarithms are to base 2, by the hardware's functions,
// whose rounding is no larger than that of the scaled ones; in FP64 one Newton step on
// log x (kFracTerms terms, ratios rt) follows.  (FP32, rms error of the jump
// against 64 bits at alpha = 0.1, 0.4, 1, 1.6, 1.9: omega in the lower half 9.9e-7,
// 2.3e-7, 1.2e-7, 1.2e-7, 1.3e-7, in the upper 5.5e-8 .. 2.8e-8; with a linear table, a
// Newton step of 26 terms and natural logarithms 1.0e-6, 3.0e-7, 1.6e-7, 1.3e-7, 1.5e-7
// and 6.2e-8 .. 1.2e-7.)
__device__ __forceinline__ float ibeta_inv_log(float y, float, float ip, float lpb, float xs, const float *cub, const float *)
{
    const float z0 = (__builtin_amdgcn_logf(y) + lpb) * ip;
    const float f = __builtin_amdgcn_exp2f(z0) * xs;
    const int i = min((int)f, kFracTab - 1);
    const float w = f - (float)i, *c = cub + 4 * i;
    const float z = z0 + fmaf(fmaf(fmaf(c[3], w, c[2]), w, c[1]), w, c[0]);
    return f < (float)kFracTab ? fminf(z, -1.f) : -1.f;
}
__device__ __forceinline__ double ibeta_inv_log(double y, double p, double ip, double lpb, double xs, const double *cub,
                                                const double *rt)
{
    const double lhalf = -0.69314718055994530942;
    const double ly = log(y);
    const double z0 = (ly + lpb) * ip;
    const double f = exp(z0) * xs;
    const int i = min((int)f, kFracTab - 1);
    const double w = f - (double)i, *c = cub + 4 * i;
    double z = z0 + fma(fma(fma(c[3], w, c[2]), w, c[1]), w, c[0]);
    z = f < (double)kFracTab && z < lhalf ? z : lhalf;
    const double x = exp(z);
    double S = 1.0, t = 1.0;
#pragma unroll
    for (int k = 0; k < kFracTerms; ++k) {
        t *= x * rt[k];
        S += t;
    }
    const double lI = p * z + (1.0 - p) * log1p(-x) - lpb + log(S);
    z = z - (lI - ly) * (1.0 - x) * S / p;
    return z < lhalf ? z : lhalf;
}

// 1 / sqrt(t) for t in [1/2, 1]
__device__ __forceinline__ double inv_sqrt(double t) { return 1.0 / sqrt(t); }
__device__ __forceinline__ float inv_sqrt(float t)
{
    const float y = __builtin_amdgcn_rsqf(t);   // one Newton step takes its last bit's error away
    return fmaf(0.5f * y, fmaf(-(t * y), y, 1.f), y);
}

// the inverse of the logarithm that ibeta_inv_log takes
__device__ __forceinline__ double log_exp(double x) { return exp(x); }
__device__ __forceinline__ float log_exp(float x) { return __builtin_amdgcn_exp2f(x); }

// (1 - x^2)^a, |x| < 1.  FP32 by the hardware's functions: against 64 bits over 2^20 points
// the rms error is 1-4% below the library's expf(a logf) at a = 0.05 .. 0.95.
__device__ __forceinline__ double frac_weight(double x, double a) { return exp(a * log((1.0 - x) * (1.0 + x))); }
__device__ __forceinline__ float frac_weight(float x, float a)
{
    return __builtin_amdgcn_exp2f(a * __builtin_amdgcn_logf((1.f - x) * (1.f + x)));
}

// sin x for |x| < 1 by its Taylor series, the next term below 2^-32 (FP32) or 2^-56 of x
// (FP32: rms error 1.31e-8, the library's 1.40e-8)
template <typename T>
__device__ __forceinline__ T sin_unit(T x)
{
    const T x2 = x * x;
    T s = (T)0;
    if constexpr (sizeof(T) == 8) {
        s = m_fma(s, x2, (T)(1.0 / 355687428096000.0));
        s = m_fma(s, x2, (T)(-1.0 / 1307674368000.0));
        s = m_fma(s, x2, (T)(1.0 / 6227020800.0));
    }
    s = m_fma(s, x2, (T)(-1.0 / 39916800.0));
    s = m_fma(s, x2, (T)(1.0 / 362880.0));
    s = m_fma(s, x2, (T)(-1.0 / 5040.0));
    s = m_fma(s, x2, (T)(1.0 / 120.0));
    s = m_fma(s, x2, (T)(-1.0 / 6.0));
    return m_fma(x * x2, s, x);
}

// one inverse per lane whichever half of (0,1) omega falls in: x <= 1/2 solves
// I_x(a, 1-a) = omega for log x; otherwise z = 1 - x solves I_z(1-a, a) = 1 - omega
// for log z.
template <typename T>
__device__ __forceinline__ T frac_jump(const Physics &ph, T R, T om, const T *tl)
{
    constexpr double base = sizeof(T) == 8 ? 1.0 : 1.4426950408889634074;   // 1 / log of the base
    const T a = (T)ph.frac_a;
    const bool lower = om <= (T)ph.frac_half;
    const T *rt = tl + 2 * 4 * kFracTab;
    const T z = ibeta_inv_log(lower ? om : (T)1 - om, lower ? a : (T)1 - a,
                              lower ? (T)(1.0 / ph.frac_a) : (T)(1.0 / (1.0 - ph.frac_a)),
                              lower ? (T)(base * ph.frac_lpb1) : (T)(base * ph.frac_lpb2),
                              lower ? (T)ph.frac_xs[0] : (T)ph.frac_xs[1], tl + (lower ? 0 : 4 * kFracTab),
                              rt + (lower ? 0 : kFracTerms));
    const T e = log_exp(lower ? (T)-0.5 * z : z);
    return R * (lower ? e : inv_sqrt((T)1 - e));
}

constexpr int kFracRow = 2 * ((kMaxP + 3) / 4 * 4);   // most entries of a slab row

// a lane's value, the same for the whole wave
__device__ __forceinline__ float lane_value(float x, int lane)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane));
}
__device__ __forceinline__ double lane_value(double x, int lane)
{
    const uint64_t b = __double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
    return __longlong_as_double((int64_t)((uint64_t)hi << 32 | lo));
}

// Bound by vector instructions (two logarithms, three exponentials and the two series a
// step; 270 a wave and step).  A wave takes items of 64 paths by itself and meets no
// barrier: the step's slab row comes through the wave's own part of LDS, loaded a step
// ahead, the tables of the recurrence as scalar operands, and the source's time factors
// from the lanes of a 64-step window.  Launches of 540672 paths at n = 11, alpha = 0.4,
// FP32: 116 us.  (A block barrier each step, tables read from LDS, 40 source terms, a
// Newton step of 26 terms and items from a counter took 433 us; with the steps as now but
// the counter and one line of statistics, whose atomics are served one by one, 244.)
// SRC: the source kind, 5 .. 7, or 0 (none), compiled apart: fewer uniform operands spill.
template <typename T, int SRC>
__global__ void __launch_bounds__(256) frac_advance_kernel(RoundArgs a)
{
    extern __shared__ u32x4 lds[];
    const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wave = (int)uniform_u32(tid >> 6);
    const Physics &ph = a.phys;
    const int PP = a.PP, kmax = ph.frac_kmax;   // multiples of 4; slab rows and tables hold zeros past their terms
    cptr<T> tA = as_const((const T *)ph.frac_tab), tC = tA + kmax, tlam = tC + kmax, tsrc = tlam + kmax;
    T *tl = (T *)lds;   // the cubics and the series ratios, looked up by lane, then the waves' slab rows
    T *S = tl + 2 * 4 * kFracTab + 2 * ph.frac_nt + wave * kFracRow;
    {
        const T *src = (const T *)ph.frac_tab + 4 * kmax;
        for (int i = tid; i < 2 * 4 * kFracTab + 2 * ph.frac_nt; i += blockDim.x) tl[i] = src[i];
    }
    __syncthreads();
    cptr<GroupDesc> groups = as_const(a.groups);
    cptr<NodeDesc> nodes = as_const(a.nodes);
    const int64_t total = a.batch_prefix[a.n_groups];
    unsigned long long evals = 0, slots = 0;
    using State = PathState<T, 1>;
    const State *sin = (const State *)a.state_in;
    State *sout = (State *)a.state_out;
    const T fa = (T)ph.frac_a;

    // A group's items take the same time, N* steps, and the last groups' the most: dealt
    // out from the last one down, back and forth over the grid's waves (no counter: its
    // atomics, 9 ns each, would take as long as the walks).  The rotation by 256 blocks,
    // one of a compute unit's, gives each SIMD items from all over the order.
    const int64_t grid = (int64_t)gridDim.x * nw;
    const int64_t self = (int64_t)((wave + blockIdx.x / 256) % nw) * gridDim.x + blockIdx.x;
    for (int64_t pass = 0; pass * grid < total; ++pass) {
        const int64_t taken = pass * grid + (pass & 1 ? grid - 1 - self : self);
        if (taken >= total) continue;
        const int64_t item = total - 1 - taken;
        int lo = 0, hi = a.n_groups - 1;   // last g with batch_prefix[g] <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.batch_prefix[mid] <= item) lo = mid; else hi = mid - 1;
        }
        const int g = (int)uniform_u32(lo);
        const int64_t b = item - a.batch_prefix[g];
        cptr<GroupDesc> G = groups + g;
        const int nstar = G->nstar;
        const int q0 = a.round * a.steps;
        const int q1 = min(q0 + a.steps, nstar);
        const T delta = (T)G->delta, R = (T)G->jump;
        const double span = G->span, t_prev = G->t_prev, ddelta = G->delta;
        const uint32_t c3 = G->c3 | (uint32_t)a.tag;
        const int64_t live = a.round == 0 ? (int64_t)G->node_count * a.mcount : (int64_t)a.live_in[g];
        const T *gtab = (const T *)a.slab_table + G->slab;
        // the slab row of a step: loaded a step ahead, one or two values a lane, and read
        // back as broadcasts from the wave's own part of LDS
        T row0 = (T)0, row1 = (T)0;
        const auto load_row = [&](int qq) {
            const T *src = gtab + (int64_t)qq * a.slab_stride;
            if (lane < 2 * PP) row0 = src[lane];
            if (lane + 64 < 2 * PP) row1 = src[lane + 64];
        };
        load_row(q0);

        T X = (T)0, acc = (T)0, comp = (T)0;
        uint32_t node = 0, sample = 0, c0 = 0;
        const int64_t p = b * 64 + lane;
        bool alive = p < live;
        if (alive) {
            if (a.round == 0) {
                node = (uint32_t)(G->node_begin + p / a.mcount);
                sample = (uint32_t)(a.m0 + p % a.mcount);
                X = (T)nodes[node].x0[0];
            } else {
                const State st = sin[G->path_off + p];
                X = st.x[0];
                acc = st.acc;
                comp = st.comp;
                node = st.node;
                sample = st.sample;
            }
            c0 = nodes[node].c0;
        }
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        T tt = (T)0, tp = (T)0;   // T(tau), T'(tau) of the manufactured source at step q0 + 64 i + lane
        int q = q0;
        for (; q < q1; ++q) {
            const int slot = (q - q0) & 63;
            if (SRC > 0 && slot == 0) {
                const T tau = (T)(t_prev + (span - (double)(q + lane) * ddelta));
                if (q + lane >= q1) {
                    tt = tp = (T)0;
                } else if (SRC == 5) {
                    const T qd = (T)1 + tau * tau;
                    tt = m_exp(m_cos(tau)) / qd;
                    tp = tt * (-m_sin(tau) - (T)2 * tau / qd);
                } else if (SRC == 6) {
                    const T rho = (T)ph.src_param[0];
                    tt = m_exp(rho * m_log(tau));
                    tp = rho * tt / tau;
                } else {
                    tt = (T)1 + (T)ph.src_param[3] * tau;
                    tp = (T)ph.src_param[3];
                }
            }
            const T Tt = lane_value(tt, slot), Tp = lane_value(tp, slot);
            if (lane < 2 * PP) S[lane] = row0;
            if (lane + 64 < 2 * PP) S[lane + 64] = row1;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (q + 1 < q1) load_row(q + 1);
            bool any_live = false;
            if (alive) {
                if ((q & 1) == 0 || q == q0) {
                    uint32_t k0 = a.key0, k1 = a.key1;
                    asm volatile("" : "+s"(k0), "+s"(k1));   // the rounds' keys are formed here, not kept (and spilled)
                    philox(c0, sample, (uint32_t)(q >> 1), c3, k0, k1, w);
                }
                const uint32_t wo = (q & 1) ? w[2] : w[0], ws = (q & 1) ? w[3] : w[1];
                const T J = frac_jump<T>(ph, R, u01(wo, (T)0), tl);
                const T Y = m_fma(J, (ws & 1u) ? (T)1 : (T)-1, X);
                if (!(fabs(Y) < (T)1)) {   // path ended: L = q (its value is stored with the others')
                    alive = false;
                } else {
                    // ---- residual at X_q, tau_q = t_{n,l} - q Delta
                    const T wgt = frac_weight(X, fa);
                    T pm = (T)0, pc = (T)1, uj = (T)0, vj = (T)0, F = (T)0, Gs = (T)0;
                    // (A x) p, not A (x p): its rms error over 16 modes is 5 .. 10% smaller, and A x
                    // is off the chain from mode to mode
                    const auto next = [&](int k) {
                        const T pn = m_fma(tA[k] * X, pc, -(tC[k] * pm));
                        pm = pc;
                        pc = pn;
                    };
                    for (int k = 0; k < PP; k += 4) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            uj = m_fma(S[k + j], pc, uj);
                            vj = m_fma(S[PP + k + j], pc, vj);
                            F = m_fma(S[k + j], tlam[k + j] * pc, F);
                            if constexpr (SRC > 0) Gs = m_fma(tsrc[k + j], pc, Gs);
                            next(k + j);
                        }
                    }
                    for (int k = PP; SRC > 0 && k < kmax; k += 4) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            Gs = m_fma(tsrc[k + j], pc, Gs);
                            next(k + j);
                        }
                    }
                    // manufactured source s = w g T' + T (-Delta)^{alpha/2}(w g) - f(w g T)
                    T src = (T)0;
                    if constexpr (SRC > 0) {
                        T gx;
                        if (SRC == 5)
                            gx = sin_unit(X);
                        else if (SRC == 6)
                            gx = m_cos(X * X * X + (T)1) / ((T)10 * X * X + (T)1);
                        else
                            gx = (T)ph.src_param[0] + X * ((T)ph.src_param[1] + X * (T)ph.src_param[2]);
                        src = wgt * gx * Tp + Gs * Tt - f_of<T>(ph, wgt * gx * Tt);
                    }
                    // Picard form (eq. uast): the integrand f(u*) + s only
                    const T r = ph.picard ? f_of<T>(ph, wgt * uj) + src : f_of<T>(ph, wgt * uj) + src + wgt * vj - F;
                    const T y = delta * r;
                    if constexpr (sizeof(T) == 4) {
                        const T yc = y - comp;
                        const T ta = acc + yc;
                        comp = (ta - acc) - yc;
                        acc = ta;
                    } else {
                        acc += y;
                    }
                    X = Y;
                    ++evals;
                    any_live = true;
                }
            }
            ++slots;
            if (__ballot(any_live) == 0ull) { ++q; break; }
        }

        // ---- Picard form (eq. uast): a path still inside after all N* steps adds
        // the interval's initial data u*(X_{N*}, t_{n-1}), the slab of step N*
        if (ph.picard && q1 == nstar && q == q1 && alive) {
            const T *Sn = gtab + (int64_t)nstar * a.slab_stride;
            T pm = (T)0, pc = (T)1, uj = (T)0;
            for (int k = 0; k < a.P; ++k) {
                uj = m_fma(Sn[k], pc, uj);
                const T pn = m_fma(tA[k] * X, pc, -(tC[k] * pm));
                pm = pc;
                pc = pn;
            }
            const T y = frac_weight(X, fa) * uj;
            if constexpr (sizeof(T) == 4) {
                const T yc = y - comp;
                const T ta = acc + yc;
                comp = (ta - acc) - yc;
                acc = ta;
            } else {
                acc += y;
            }
        }

        // ---- paths ended in this round or at N* (a store for each end, with its wait, in
        // the steps made them twice as long), and those carried to the next round
        const bool carry = alive && q1 < nstar;
        if (p < live && !carry)
            a.result[(int64_t)nodes[node].out * a.mcount + (sample - a.m0)] = (double)acc - (double)comp;
        const unsigned long long mask = __ballot(carry);
        if (mask != 0ull) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(a.live_out + g, (uint32_t)__popcll(mask));
            base = __shfl(base, 0, 64);
            if (carry) {
                const uint32_t off = base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                State st;
                st.x[0] = X;
                st.acc = acc;
                st.comp = comp;
                st.node = node;
                st.sample = sample;
                sout[G->path_off + off] = st;
            }
        }
    }
    add_stats(a, evals, slots);
}

// dynamic LDS of the fractional round kernel: the cubics, the series ratios, a slab row per wave (at most 16)
size_t frac_lds_bytes(int fp32)
{
    return fp32 ? (size_t)(2 * 4 * kFracTab + 16 * kFracRow) * 4 : (size_t)(2 * 4 * kFracTab + 2 * kFracTerms + 16 * kFracRow) * 8;
}

template <typename T>
static hipError_t frac_launch(const RoundArgs &a, dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    switch (a.phys.src_kind) {
    case 5: hipLaunchKernelGGL((frac_advance_kernel<T, 5>), grid, block, lds, s, a); break;
    case 6: hipLaunchKernelGGL((frac_advance_kernel<T, 6>), grid, block, lds, s, a); break;
    case 7: hipLaunchKernelGGL((frac_advance_kernel<T, 7>), grid, block, lds, s, a); break;
    default: hipLaunchKernelGGL((frac_advance_kernel<T, 0>), grid, block, lds, s, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_adv_frac(const RoundArgs &a, int fp32, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t s)
{
    if (a.phys.dim != 1 || a.batch != 64 || a.P > a.PP || a.PP % 4 || a.phys.frac_kmax % 4 || a.phys.frac_kmax < a.PP ||
        a.phys.frac_nt != (fp32 ? 0 : kFracTerms) || lds_bytes < frac_lds_bytes(fp32))
        return hipErrorInvalidValue;
    return fp32 ? frac_launch<float>(a, grid, block, lds_bytes, s) : frac_launch<double>(a, grid, block, lds_bytes, s);
}

}  // namespace hpsmc
