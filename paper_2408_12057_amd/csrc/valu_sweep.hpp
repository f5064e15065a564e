// valu_sweep.hpp -- annealing sweeps for the closed-form targets (isotropic
// Gaussian, equal-weight Gaussian mixture) with RWMH, MALA and HMC moves.
//
// These paths are bound by plain VALU arithmetic (Philox rounds, binary64
// Box-Muller, distance and gradient sums), so the design keeps each particle in
// registers: a particle occupies LPP adjacent lanes, each holding DPL of its
// coordinates (fp32 state, binary64 arithmetic).  Per-particle scalars (ell,
// log w, log alpha) are reduced over the LPP lanes with a butterfly so every
// lane of the group holds the same bits and takes the same MH decision.
//
// Two drivers share the particle code:
//  * k_oais_valu -- the AIS case with the particle loop outside the time loop
//    (Sec. "Optimised AIS"): a wave owns a tile of 64/LPP particles for all T
//    steps; the moments g_hat_{t,i} (eq. CESS) are streamed into a fixed number
//    of slots S of O(T) memory each, independent of N and of the grid shape.
//  * k_asmc_step / k_asmc_merge / resampler -- the adaptive-resampling case
//    (Alg. 1 with AR): one launch per step t, state in HBM, a two-level merge
//    in one launch that evaluates the trigger on the device, and the
//    integer-CDF systematic resampler (launched every step, does nothing
//    unless the trigger fired).
#pragma once
#include "kernels.hpp"
#include "normal_math.hpp"

namespace oasmc {



__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Precomputed reference/target scalars.
struct Consts {
    double half_inv_s2r;  // 1 / (2 ref_sigma2)
    double inv_s2r;       // 1 / ref_sigma2
    double cst_eta;       // (d/2) log(2 pi ref_sigma2)
    double sref;          // sqrt(ref_sigma2)
    double half_inv_s2;   // Gaussian target: 1/(2 sigma2)
    double inv_s2;        // Gaussian target: 1/sigma2
    double logK;
};

__device__ __forceinline__ Consts make_consts(const TargetDev& tg)
{
    Consts c;
    c.inv_s2r = 1.0 / tg.ref_sigma2;
    c.half_inv_s2r = 0.5 / tg.ref_sigma2;
    c.cst_eta = 0.5 * tg.d * (1.8378770664093454835606594728112 + log(tg.ref_sigma2));
    c.sref = sqrt(tg.ref_sigma2);
    c.half_inv_s2 = 0.5 / tg.sigma2;
    c.inv_s2 = 1.0 / tg.sigma2;
    c.logK = log((double)(tg.K > 0 ? tg.K : 1));
    return c;
}

// Target parameters staged in LDS: reference mean [d], then the Gaussian mean
// [d] or the mixture means [K*d], then the mixture 1/(2 v_k), 1/v_k (the view
// type ParView is declared in kernels.hpp); the caller's barrier publishes them.

__device__ __forceinline__ ParView stage_params(const TargetDev& tg, char* sh)
{
    const int d = tg.d;
    const int nmu = (tg.family == kGmm) ? tg.K * d : d;
    double* hv = reinterpret_cast<double*>(sh);
    double* iv = hv + kMaxK;
    float* m = reinterpret_cast<float*>(iv + kMaxK);
    float* mu = m + d;
    for (int i = threadIdx.x; i < d; i += blockDim.x) m[i] = tg.ref_mean ? tg.ref_mean[i] : 0.f;
    const float* src = (tg.family == kGmm) ? tg.means : tg.mu;
    if (src)
        for (int i = threadIdx.x; i < nmu; i += blockDim.x) mu[i] = src[i];
    // 1/(2 v_k), 1/v_k; zero beyond K (padded components of a block)
    for (int k = threadIdx.x; k < kMaxK; k += blockDim.x) {
        const bool on = tg.family == kGmm && k < tg.K;
        const double v = on ? exp(2.0 * (double)tg.log_scales[k]) : 1.0;
        hv[k] = on ? 0.5 / v : 0.0;
        iv[k] = on ? 1.0 / v : 0.0;
    }
    return ParView{m, mu, hv, iv, nullptr, nullptr, nullptr, nullptr};
}


// The same staging followed by the binary64 lane-layout means lm, lmu of the
// move's shape (LPP, DPL) and, for kernels that draw, the tables of the normals.
template <int MOVE, int LPP, int DPL>
__device__ __forceinline__ ParView stage_params_lanes(const TargetDev& tg, char* sh, NormalTables* nt)
{
    if (nt) stage_tables(*nt);
    const ParView base = stage_params(tg, sh);
    double* lane = reinterpret_cast<double*>(sh + ((lane_params_offset(tg) + 15) & ~(size_t)15));
    const int nl = (int)lane_param_doubles(tg, LPP, DPL);
    float* lmf = nullptr;
    if (lane_param_floats(tg, MOVE, LPP, DPL) > 0) lmf = reinterpret_cast<float*>(lane + nl);
    for (int e = threadIdx.x; e < nl; e += blockDim.x) {
        const double v = lane_param(tg, LPP, DPL, e);
        lane[e] = v;
        // element (k, j, r) of the targets' means, transposed (its source is binary32)
        const int ke = e - LPP * DPL;
        if (lmf && ke >= 0) {
            const int k = ke / (LPP * DPL), j = ke / LPP % DPL, r = ke % LPP;
            lmf[(k * LPP + r) * DPL + j] = (float)v;
        }
    }
    __syncthreads();
    return ParView{base.m, base.mu, base.hiv, base.iv, lane, lane + LPP * DPL, nt, lmf};
}


// Trajectories of a tile that go without looking for near components: none while
// looking finds few, then 1, 3, 7 and at most 15 after each look in vain (the
// number left in the low four bits, the last length above them).  A look costs
// about a third of an evaluation.  Mixtures of 8 components at d = 100, 24 steps of 5
// leapfrog steps, N = 20011: overlapping 1.49 ms without looking, 1.59 with a look a
// trajectory, 1.53 so; far apart 1.56, 0.85 and 0.87.
__device__ __forceinline__ int look_in_vain(int wait)
{
    const int n = min(2 * (wait >> 4) + 1, 15);
    return (n << 4) | n;
}

// ---------------------------------------------------------------------------
// Particle arithmetic for one lane group.
// ---------------------------------------------------------------------------
// Coordinates of a lane beyond d (the tail of the last lanes' slices) hold
// exact zeros in x, z, the momentum and the gradient, and the lane-layout
// means are zero there too, so every coordinate loop runs without a branch:
// a padded coordinate adds +0 to each sum and stays +0 through every move.
template <int FAM, int LPP, int DPL>
struct Particle {
    static constexpr bool kLooks = FAM == kGmm && LPP > 1;  // HMC looks for near components
    // Mixtures over lanes of 16 coordinates have no registers left in a trajectory, see
    // mixture_multilane.
    static constexpr bool kRoomy = !kLooks || DPL <= 8;

    // reference mean and target mean k at this lane's coordinate j
    static __device__ __forceinline__ double ref(const ParView& pv, int r, int j)
    {
        return pv.lm[j * LPP + r];
    }
    static __device__ __forceinline__ double mean(const ParView& pv, int k, int r, int j)
    {
        return pv.lmu[(k * DPL + j) * LPP + r];
    }
    // The view with an offset the compiler cannot see through (always zero):
    // the means are then re-read from LDS at each evaluation instead of being
    // hoisted out of the time and leapfrog loops into registers, which for
    // K d / LPP beyond a few dozen would spill.
    static __device__ __forceinline__ ParView fresh(const ParView& pv)
    {
        int z0;
        asm volatile("s_mov_b32 %0, 0" : "=s"(z0));
        ParView v = pv;
        v.lm = pv.lm + z0;
        v.lmu = pv.lmu + z0;
        if (pv.lmf) v.lmf = pv.lmf + z0;
        return v;
    }

    // Inside the support (0, box)^2 of the uniform reference (kUnid).
    static __device__ __forceinline__ bool unid_inside(const TargetDev& tg, const float (&x)[DPL])
    {
        return x[0] > 0.f && (double)x[0] < tg.box && x[1] > 0.f && (double)x[1] < tg.box;
    }

    // The coordinates in binary64; in the flat evaluation, where a lane has the
    // registers, behind an empty asm: converted once and kept, where the compiler would
    // convert them again at each component.
    template <bool FLAT>
    static __device__ __forceinline__ void widen(const float (&x)[DPL], double (&xd)[DPL])
    {
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            xd[j] = (double)x[j];
            if constexpr (FLAT && kRoomy) asm("" : "+v"(xd[j]));
        }
    }

    // |x - m_ref|^2 over the particle's lanes.
    template <typename X>
    static __device__ __forceinline__ double ref_square(const ParView& pv, int r, const X (&x)[DPL])
    {
        double sse = 0.0;
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            const double b = (double)x[j] - ref(pv, r, j);
            sse = fma(b, b, sse);
        }
        return group_sum<LPP>(sse);
    }

    // ell(x) = log gamma(x) - log eta(x); with GRAD also its gradient on this
    // lane's coordinates.  r = lane index inside the group.
    // few (mixtures over several lanes): in, whether to look for the components
    // that matter; out, whether they were few.
    // value: whether ell itself is wanted (else 0 comes back: within a trajectory
    // only the gradient is, and the sums over the lanes and the logarithm are not
    // formed).
    // FLAT: see mixture_multilane.
    template <bool GRAD, bool FLAT = false>
    static __device__ __forceinline__ double eval(const TargetDev& tg, const Consts& c,
                                                  const ParView& pv0, int r, const float (&x)[DPL],
                                                  double (&g)[DPL], bool* few = nullptr,
                                                  bool value = true)
    {
        const ParView pv = fresh(pv0);
        if constexpr (FAM == kUnid) {
            // d = 2 on one lane: the log-likelihood ratio of Binomial(k | n, x y)
            // against its maximum, log1p forms near the ridge x y = k / n
            (void)r;
            (void)c;
            const double x0 = (double)x[0], x1 = (double)x[1];
            const double u = x0 * x1;
            if (GRAD) {
#pragma unroll
                for (int j = 0; j < DPL; ++j) g[j] = 0.0;
            }
            if (!unid_inside(tg, x) || !(u > 0.0 && u < 1.0)) return -INFINITY;
            const double n = tg.binom_n, k = tg.binom_k, p = k / n;
            return k * log1p((u - p) / p) + (n - k) * log1p(-(u - p) / (1.0 - p));
        } else if constexpr (FAM == kGauss) {
            double ssg = 0.0, sse = 0.0;
            if (GRAD && !value) {
#pragma unroll
                for (int j = 0; j < DPL; ++j) {
                    const double xv = (double)x[j];
                    const double a = xv - mean(pv, 0, r, j);
                    const double b = xv - ref(pv, r, j);
                    g[j] = -a * c.inv_s2 + b * c.inv_s2r;
                }
                return 0.0;
            }
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                const double xv = (double)x[j];
                const double a = xv - mean(pv, 0, r, j);
                const double b = xv - ref(pv, r, j);
                ssg = fma(a, a, ssg);
                sse = fma(b, b, sse);
                if (GRAD) g[j] = -a * c.inv_s2 + b * c.inv_s2r;
            }
            const double part = -ssg * c.half_inv_s2 + sse * c.half_inv_s2r;
            return group_sum<LPP>(part) + c.cst_eta;
        } else {
            // equal-weight mixture of unnormalised isotropic components, streamed
            // over k with a running maximum (log-sum-exp and responsibilities)
            if constexpr (LPP > 1) {
                if constexpr (GRAD) {
                    uint32_t near;
                    if (few && *few && (*few = near_components(tg, pv, r, x, near)))
                        return mixture_few<FLAT>(tg, c, pv, r, x, g, near, value);
                }
                return mixture_multilane<GRAD, FLAT>(tg, c, pv, r, x, g, value);
            }
            const double sse = value ? ref_square(pv, r, x) : 0.0;
#pragma unroll
            for (int j = 0; j < DPL; ++j)
                if (GRAD) g[j] = 0.0;
            double mx = -INFINITY, s = 0.0;
#pragma unroll 1
            for (int k = 0; k < tg.K; ++k) {
                double sq = 0.0;
#pragma unroll
                for (int j = 0; j < DPL; ++j) {
                    const double a = (double)x[j] - mean(pv, k, r, j);
                    sq = fma(a, a, sq);
                }
                const double ek = -group_sum<LPP>(sq) * pv.hiv[k];
                double wk;
                if (ek > mx) {
                    const double sc = exp(mx - ek);  // 0 on the first component
                    s *= sc;
                    if (GRAD) {
#pragma unroll
                        for (int j = 0; j < DPL; ++j) g[j] *= sc;
                    }
                    mx = ek;
                    wk = 1.0;
                } else {
                    wk = exp(ek - mx);
                }
                s += wk;
                if (GRAD) {
                    const double f = wk * pv.iv[k];
#pragma unroll
                    for (int j = 0; j < DPL; ++j)
                        g[j] = fma(f, mean(pv, k, r, j) - (double)x[j], g[j]);
                }
            }
            const double lse = value ? mx + log(s) - c.logK : 0.0;
            if (GRAD) {
                const double inv_s = 1.0 / s;
#pragma unroll
                for (int j = 0; j < DPL; ++j)
                    g[j] = g[j] * inv_s + ((double)x[j] - ref(pv, r, j)) * c.inv_s2r;
            }
            return lse + sse * c.half_inv_s2r + c.cst_eta;
        }
    }

    // The mixture term for a particle spread over LPP > 1 lanes, in two
    // passes: the exponents e_k = -|x - m_k|^2 / (2 v_k) (summed over the
    // lanes, so every lane holds them all), their maximum M, then one
    // exponential per component, computed by the lane k mod LPP only, and
    // log sum_k exp(e_k - M); the gradient gathers the weights from their
    // lanes.  (Streaming over k on every lane would repeat each exponential
    // LPP times.)
    // FLAT: the components' loops unrolled, and where a lane has the registers (8
    // coordinates or fewer) the coordinates converted once instead of at each use and
    // the gradient's components in whole blocks without branches.  For the
    // trajectories of the sweeps, whose two waves per SIMD leave registers: 24 HMC steps
    // of 5 leapfrog steps of 20011 overlapping particles, d = 100, 8 components, 1.78 ->
    // 1.53 ms; 3 leapfrog steps of 70000 at d = 30, 2.04 -> 1.65 ms.  The per-step kernel's three
    // waves spill (12.4 -> 15.1 ms for 96 steps of 65536 particles).  A MALA step, one
    // evaluation, gains with lanes of 16 coordinates in the sweeps (16 steps of 60000
    // particles, 16 components, d = 50 1.19 -> 0.91 ms), loses in the per-step kernel
    // (d = 200, N = 30000 2.28 -> 2.87 ms) and with fewer coordinates (5 to 12%).
    template <bool GRAD, bool FLAT>
    static __device__ __forceinline__ double mixture_multilane(const TargetDev& tg, const Consts& c,
                                                               const ParView& pv, int r,
                                                               const float (&x)[DPL],
                                                               double (&g)[DPL], bool value)
    {
        double xd[DPL];
        widen<FLAT>(x, xd);
        const double sse = value ? ref_square(pv, r, xd) : 0.0;
#pragma unroll
        for (int j = 0; j < DPL; ++j)
            if (GRAD) g[j] = 0.0;
        constexpr int KO = (kMaxK + LPP - 1) / LPP;  // components owned by a lane
        const int K = tg.K;
        double eo[KO];
#pragma unroll
        for (int q = 0; q < KO; ++q) eo[q] = -INFINITY;
        // exponents in blocks of kKBlock components without a branch inside a
        // block, so the independent distance chains and reductions of a block
        // interleave; the lane layout and 1/(2 v_k) are zero-padded to whole
        // blocks and a padded component gets e_k = -inf (weight 0)
        double M = -INFINITY;
        auto block = [&](int k0) {
            double sq[kKBlock];
#pragma unroll
            for (int u = 0; u < kKBlock; ++u) {
                sq[u] = 0.0;
#pragma unroll
                for (int j = 0; j < DPL; ++j) {
                    const double a = xd[j] - mean(pv, k0 + u, r, j);
                    sq[u] = fma(a, a, sq[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < kKBlock; ++u) {
                const int k = k0 + u;
                double ek = -group_sum<LPP>(sq[u]) * pv.hiv[k];
                if (k >= K) ek = -INFINITY;
                M = fmax(M, ek);
#pragma unroll
                for (int q = 0; q < KO; ++q)
                    if (k == q * LPP + r) eo[q] = ek;
            }
        };
        if constexpr (FLAT) {
#pragma unroll
            for (int k0 = 0; k0 < kMaxK; k0 += kKBlock)
                if (k0 < K) block(k0);
        } else {
#pragma unroll 1
            for (int k0 = 0; k0 < K; k0 += kKBlock) block(k0);
        }
        double wo[KO];
        double so = 0.0;
#pragma unroll
        for (int q = 0; q < KO; ++q) {
            wo[q] = (q * LPP + r < K) ? exp(eo[q] - M) : 0.0;
            so += wo[q];
        }
        const double s = group_sum<LPP>(so);
        const double lse = value ? M + log(s) - c.logK : 0.0;
        if (GRAD) {
            const int base = (int)(threadIdx.x & (kWave - 1)) & ~(LPP - 1);
            auto pull = [&](int k) {
                double w = wo[0];
#pragma unroll
                for (int q = 1; q < KO; ++q) w = (k / LPP == q) ? wo[q] : w;
                const double f = __shfl(w, base + k % LPP, kWave) * pv.iv[k];
#pragma unroll
                for (int j = 0; j < DPL; ++j)
                    g[j] = fma(f, mean(pv, k, r, j) - xd[j], g[j]);
            };
            int k1 = 0;  // components taken
            if constexpr (FLAT && kRoomy) {
#pragma unroll
                for (int k0 = 0; k0 < kMaxK; k0 += kKBlock)
                    if (k0 + kKBlock <= K) {
#pragma unroll
                        for (int u = 0; u < kKBlock; ++u) pull(k0 + u);
                    }
                k1 = K / kKBlock * kKBlock;
            }
            if constexpr (FLAT && !kRoomy) {
#pragma unroll
                for (int k = 0; k < kMaxK; ++k)
                    if (k < K) pull(k);
            } else {
#pragma unroll 1
                for (int k = k1; k < K; ++k) pull(k);
            }
            const double inv_s = 1.0 / s;
#pragma unroll
            for (int j = 0; j < DPL; ++j)
                g[j] = g[j] * inv_s + (xd[j] - ref(pv, r, j)) * c.inv_s2r;
        }
        return lse + sse * c.half_inv_s2r + c.cst_eta;
    }

    // The components whose weight relative to the largest may be above zero in
    // binary64 (bits of `near`, the same on the particle's lanes), from distances
    // in binary32: half the issue cycles of the binary64 ones, and sums over the lanes
    // that leave each lane its own components (13 instructions for four, against 32
    // for sums that every lane holds, and the comparison is made once).  States and means are binary32, so a difference is
    // off by 2^-24 of itself and a distance, its scaling and the comparison by
    // less than 64 such roundings (4e-6); exp underflows to zero below -746.  A
    // component whose distance or exponent is not finite in binary32 is kept.  False
    // when some particle of the wave has more than half the components near, or three
    // eighths on two lanes a particle, where 32 particles share the walk (4 of 8 near,
    // 24 steps: d = 30, N = 70000 1.93 ms by the walk and 1.65 all at once, d = 100,
    // N = 20011 1.43 and 1.48).
    static __device__ __forceinline__ bool near_components(const TargetDev& tg, const ParView& pv,
                                                           int r, const float (&x)[DPL],
                                                           uint32_t& near)
    {
        constexpr int KO = (kMaxK + LPP - 1) / LPP;
        constexpr int C = LPP >= 4 ? 4 : 2;
        static_assert(kKBlock == 4, "two levels of the exchange");
        constexpr float slack = 4e-6f;
        const int K = tg.K;
        float lo = -INFINITY;  // below the largest exponent
        float hi[KO];          // above the exponents of the owned components
#pragma unroll
        for (int q = 0; q < KO; ++q) hi[q] = -INFINITY;
#pragma unroll 1
        for (int k0 = 0; k0 < K; k0 += kKBlock) {
            float sq[kKBlock];
#pragma unroll
            for (int u = 0; u < kKBlock; ++u) {
                const float4* m = reinterpret_cast<const float4*>(pv.lmf + ((k0 + u) * LPP + r) * DPL);
                sq[u] = 0.f;
#pragma unroll
                for (int jj = 0; jj < DPL / 4; ++jj) {
                    const float4 v = m[jj];
                    const float a = x[4 * jj] - v.x, b = x[4 * jj + 1] - v.y;
                    const float e = x[4 * jj + 2] - v.z, f = x[4 * jj + 3] - v.w;
                    sq[u] = fmaf(a, a, sq[u]);
                    sq[u] = fmaf(b, b, sq[u]);
                    sq[u] = fmaf(e, e, sq[u]);
                    sq[u] = fmaf(f, f, sq[u]);
                }
            }
            // sums over the lanes that leave component k0 + r mod C (and those C,
            // 2 C, .. behind it) with lane r
#pragma unroll
            for (int v = 0; v < kKBlock / 2; ++v)
                sq[v] = ((r & 1) ? sq[2 * v + 1] : sq[2 * v]) +
                        dpp_f32<kDppXor1>((r & 1) ? sq[2 * v] : sq[2 * v + 1]);
            if constexpr (C == 4) {
#pragma unroll
                for (int v = 0; v < kKBlock / 4; ++v)
                    sq[v] = ((r & 2) ? sq[2 * v + 1] : sq[2 * v]) +
                            dpp_f32<kDppXor2>((r & 2) ? sq[2 * v] : sq[2 * v + 1]);
            }
#pragma unroll
            for (int v = 0; v < kKBlock / C; ++v) {
                const int k = k0 + C * v + (r & (C - 1));
                if constexpr (LPP == 8) sq[v] += dpp_f32<kDppHalfMirror>(dpp_f32<kDppQuadRev>(sq[v]));
                if constexpr (LPP == 16) {
                    sq[v] += dpp_f32<kDppRor8>(sq[v]);
                    sq[v] += dpp_f32<kDppRor4>(sq[v]);
                }
                const float e = sq[v] * (float)pv.hiv[k];
                lo = (k < K) ? fmaxf(lo, -e * (1.f + slack)) : lo;
                // (beyond binary32 its true exponent may lie anywhere below lo)
                const float above = e < INFINITY ? -e * (1.f - slack) : INFINITY;
#pragma unroll
                for (int q = 0; q < KO; ++q)
                    if (k == q * LPP + r) hi[q] = above;
            }
        }
        lo = fmaxf(lo, dpp_f32<kDppXor1>(lo));
        if constexpr (C == 4) lo = fmaxf(lo, dpp_f32<kDppXor2>(lo));
        const int base = (int)(threadIdx.x & (kWave - 1)) & ~(LPP - 1);
        near = 0u;
#pragma unroll
        for (int q = 0; q < KO; ++q) {
            const uint64_t bal = __ballot(q * LPP + r < K && !(hi[q] < lo - 746.f - slack * fabsf(lo)));
            near |= (uint32_t)((bal >> base) & ((1u << LPP) - 1u)) << (q * LPP);
        }
        return __ballot(__popc(near) > (LPP > 2 ? K / 2 : (3 * K + 7) / 8)) == 0;
    }

    // The mixture term from the components in `near` (bits, at least one): each
    // particle walks its own, so a wave takes as many turns as its particle with
    // the most.  The others' weights are exactly zero and add nothing to any sum,
    // so the results are those of mixture_multilane bit for bit.  With the
    // components of the d = 100, 8-component target apart (one near, mostly) an
    // evaluation and leapfrog step issue about 115 binary64 instructions a wave
    // instead of 496 (96 HMC steps of 20011 particles: 6.20 -> 3.93 ms, of which
    // 4.44 -> 3.93 come from ell formed at a trajectory's end only, one force an
    // evaluation and the reduction of near_components; 3.46 ms now).
    template <bool FLAT>
    static __device__ __forceinline__ double mixture_few(const TargetDev& tg, const Consts& c,
                                                         const ParView& pv, int r,
                                                         const float (&x)[DPL], double (&g)[DPL],
                                                         uint32_t near, bool value)
    {
        double xd[DPL];
        widen<FLAT>(x, xd);
        const double sse = value ? ref_square(pv, r, xd) : 0.0;
#pragma unroll
        for (int j = 0; j < DPL; ++j) g[j] = 0.0;
        constexpr int KO = (kMaxK + LPP - 1) / LPP;
        if (__ballot((near & (near - 1u)) != 0u) == 0) {
            // one component a particle: its weight, their sum and its inverse are
            // 1, the logarithm 0 (exactly, as the functions give them).  The
            // exponent and the inverse stand behind an empty asm, so that no
            // product is fused here that the general form rounds.
            const int k = __ffs(near) - 1;
            double lse = 0.0, inv_s = 1.0;
            asm volatile("" : "+v"(inv_s));
            if (value) {
                double sq = 0.0;
#pragma unroll
                for (int j = 0; j < DPL; ++j) {
                    const double a = xd[j] - mean(pv, k, r, j);
                    sq = fma(a, a, sq);
                }
                double ek = -group_sum<LPP>(sq) * pv.hiv[k];
                asm volatile("" : "+v"(ek));
                lse = ek - c.logK;
            }
            const double f = pv.iv[k];
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                g[j] = fma(f, mean(pv, k, r, j) - xd[j], g[j]);
                g[j] = g[j] * inv_s + (xd[j] - ref(pv, r, j)) * c.inv_s2r;
            }
            return lse + sse * c.half_inv_s2r + c.cst_eta;
        }
        double eo[KO];
#pragma unroll
        for (int q = 0; q < KO; ++q) eo[q] = -INFINITY;
        double M = -INFINITY;
        for (uint32_t left = near; __ballot(left != 0u) != 0; left &= left - 1u) {
            const bool on = left != 0u;
            const int k = on ? __ffs(left) - 1 : 0;
            double sq = 0.0;
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                const double a = xd[j] - mean(pv, k, r, j);
                sq = fma(a, a, sq);
            }
            const double ek = -group_sum<LPP>(sq) * pv.hiv[k];
            if (on) M = fmax(M, ek);
#pragma unroll
            for (int q = 0; q < KO; ++q)
                if (on && k == q * LPP + r) eo[q] = ek;
        }
        const int base = (int)(threadIdx.x & (kWave - 1)) & ~(LPP - 1);
        double wo[KO];
        double so = 0.0;
        uint32_t left = 0u;  // components with weight
#pragma unroll
        for (int q = 0; q < KO; ++q) {
            wo[q] = (q * LPP + r < tg.K) ? exp(eo[q] - M) : 0.0;
            so += wo[q];
            const uint64_t bal = __ballot(!(wo[q] == 0.0));
            left |= (uint32_t)((bal >> base) & ((1u << LPP) - 1u)) << (q * LPP);
        }
        const double s = group_sum<LPP>(so);
        const double lse = value ? M + log(s) - c.logK : 0.0;
        for (; __ballot(left != 0u) != 0; left &= left - 1u) {
            const bool on = left != 0u;
            const int k = on ? __ffs(left) - 1 : 0;
            double w = wo[0];
#pragma unroll
            for (int q = 1; q < KO; ++q) w = (k / LPP == q) ? wo[q] : w;
            // (the owner's lane holds component k in the same register as here)
            const double f = __shfl(w, base + k % LPP, kWave) * pv.iv[k];
            if (on) {
#pragma unroll
                for (int j = 0; j < DPL; ++j) g[j] = fma(f, mean(pv, k, r, j) - xd[j], g[j]);
            }
        }
        const double inv_s = 1.0 / s;
#pragma unroll
        for (int j = 0; j < DPL; ++j)
            g[j] = g[j] * inv_s + (xd[j] - ref(pv, r, j)) * c.inv_s2r;
        return lse + sse * c.half_inv_s2r + c.cst_eta;
    }

    // Normals of this lane's coordinates 4 bb .. 4 bb + 3 (zero beyond d) of
    // one (particle, step, stream) sequence: block r DPL / 4 + bb of it.  With
    // one lane per particle the block index is the same in every lane, so the
    // second Box-Muller pair of a block that ends beyond d is skipped by a
    // uniform branch; with several lanes per particle the block index differs
    // across the wave, the branch would diverge (no saving) and its extra live
    // values cost the wide layouts registers, so the pair is always formed.
    static __device__ __forceinline__ void normals_block(const ParView& pv, const RngKey& key,
                                                         uint32_t n, uint32_t t, uint32_t stream,
                                                         int r, int d, int bb, double (&q)[4],
                                                         uint32_t substep = 0u)
    {
        static_assert(DPL % 4 == 0, "lane slices are whole blocks of 4 coordinates");
        const int b = r * (DPL / 4) + bb;
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = 0.0;
        // (one lane per particle: every block but the last holds coordinates in a
        // shape that fits d, and a branch around it would only keep the blocks from
        // interleaving; 2^22 particles at d = 10, 64 steps: 0.18 ms of 8)
        const bool last = bb == DPL / 4 - 1;
        if ((LPP == 1 && !last) || 4 * b < d) {
            double z[4];
            const uint4 w = draw_block(key, n, t, stream, substep, (uint32_t)b);
            box_muller(*pv.nt, w.x, w.y, z[0], z[1]);
            z[2] = z[3] = 0.0;
            if (LPP > 1 || !last || d - 4 * b > 2) box_muller(*pv.nt, w.z, w.w, z[2], z[3]);
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = (4 * b + u < d) ? z[u] : 0.0;
        }
    }

    // d normals of one (particle, step, stream) split over the group's lanes.
    static __device__ __forceinline__ void normals(const ParView& pv, const RngKey& key, uint32_t n,
                                                   uint32_t t, uint32_t stream, int r, int d,
                                                   double (&z)[DPL])
    {
#pragma unroll
        for (int bb = 0; bb < DPL / 4; ++bb) {
            double q[4];
            normals_block(pv, key, n, t, stream, r, d, bb, q);
#pragma unroll
            for (int u = 0; u < 4; ++u) z[4 * bb + u] = q[u];
        }
    }

    // X_0 ~ eta.
    static __device__ __forceinline__ double init(const TargetDev& tg, const Consts& c,
                                                  const ParView& pv, const RngKey& key, uint32_t n,
                                                  int r, float (&x)[DPL], double (&g)[DPL],
                                                  bool grad)
    {
        if constexpr (FAM == kUnid) {
            // uniform reference: coordinate i from word i of block 0
            const uint4 w = draw_block(key, n, 0u, kStreamInit, 0u, 0u);
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                x[j] = 0.f;
                g[j] = 0.0;
            }
            x[0] = (float)(tg.box * word_uniform(w.x));
            x[1] = (float)(tg.box * word_uniform(w.y));
            return eval<false>(tg, c, pv, r, x, g);
        }
        double z[DPL];
        normals(pv, key, n, 0u, kStreamInit, r, tg.d, z);
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            x[j] = (float)(ref(pv, r, j) + c.sref * z[j]);
            g[j] = 0.0;
        }
        return grad ? eval<true>(tg, c, pv, r, x, g) : eval<false>(tg, c, pv, r, x, g);
    }

    // One MH step targeting pi_beta.  Returns the accept decision (the same on
    // every lane of the group).
    template <int MOVE>
    static __device__ __forceinline__ bool move(const TargetDev& tg, const Consts& c,
                                                const ParView& pv, const RngKey& key, uint32_t n,
                                                uint32_t t, int r, int L, double beta, double eps,
                                                float (&x)[DPL], double& ell, double (&g)[DPL],
                                                int forced = -1, int* wait = nullptr)
    {
        // RWMH draws its normals block by block inside the proposal loop
        // (shorter live ranges); MALA and HMC draw them all first
        if constexpr (MOVE == kRwmh3 || FAM == kUnid) {
            // random-walk substeps (one for kRwmh, three with standard
            // deviations eps (0.1, 1, 10) for kRwmh3), each with its own
            // normals and accept uniform (counter substep j); the decision
            // reported is whether any substep was accepted
            constexpr int NS = (MOVE == kRwmh3) ? 3 : 1;
            bool any = false;
#pragma unroll
            for (int sub = 0; sub < NS; ++sub) {
                const double sd = (MOVE == kRwmh3) ? eps * (sub == 0 ? 0.1 : (sub == 1 ? 1.0 : 10.0))
                                                   : eps;
                float xq[DPL];
                double gq[DPL];
                double dle = 0.0;
#pragma unroll
                for (int bb = 0; bb < DPL / 4; ++bb) {
                    double q[4];
                    normals_block(pv, key, n, t, kStreamMove, r, tg.d, bb, q, (uint32_t)sub);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int j = 4 * bb + u;
                        xq[j] = (float)((double)x[j] + sd * q[u]);
                        if constexpr (FAM != kUnid) {
                            const double a = (double)x[j] - ref(pv, r, j);
                            const double b = (double)xq[j] - ref(pv, r, j);
                            dle += a * a - b * b;
                        }
                    }
                }
                const double ellq = eval<false>(tg, c, pv, r, xq, gq);
                double la;
                if constexpr (FAM == kUnid)
                    la = unid_inside(tg, xq) ? beta * (ellq - ell) : -INFINITY;
                else
                    la = group_sum<LPP>(dle) * c.half_inv_s2r + beta * (ellq - ell);
                const uint4 w = draw_block(key, n, t, kStreamAccept, (uint32_t)sub, 0u);
                const bool acc = (forced >= 0) ? (forced != 0) : (-0.5 * minus2_log_word(*pv.nt, w.x) < la);
                if (acc) {
#pragma unroll
                    for (int j = 0; j < DPL; ++j) x[j] = xq[j];
                    ell = ellq;
                }
                any = any || acc;
            }
            return any;
        }
        float xp[DPL];
        double gp[DPL];
        double ellp;
        const bool acc = propose<MOVE>(tg, c, pv, key, n, t, r, L, beta, eps, x, ell, g, xp, ellp, gp,
                                       forced, wait);
        if (acc) {
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                x[j] = xp[j];
                if (uses_grad(MOVE)) g[j] = gp[j];
            }
            ell = ellp;
        }
        return acc;
    }

    // The proposal of one step and its accept decision, the state as it was: what
    // becomes of both is the caller's (grad ell of a state that lies in memory is
    // dead here after the first half step).
    // FLAT: the sweeps, see mixture_multilane.  wait (HMC, mixtures over lanes, FLAT):
    // see look_in_vain; the other form looks every time (with a condition on its first
    // look the step kernel keeps 30 scalar registers more in vector lanes, 3 % of its
    // time).
    template <int MOVE, bool FLAT = true>
    static __device__ __forceinline__ bool propose(const TargetDev& tg, const Consts& c,
                                                   const ParView& pv, const RngKey& key, uint32_t n,
                                                   uint32_t t, int r, int L, double beta, double eps,
                                                   const float (&x)[DPL], double ell,
                                                   const double (&g)[DPL], float (&xp)[DPL],
                                                   double& ellp, double (&gp)[DPL], int forced = -1,
                                                   int* wait = nullptr)
    {
        double z[DPL];
        if constexpr (uses_grad(MOVE)) normals(pv, key, n, t, kStreamMove, r, tg.d, z);
        double log_alpha;
        if constexpr (MOVE == kRwmh) {
            double dle = 0.0;
#pragma unroll
            for (int bb = 0; bb < DPL / 4; ++bb) {
                double q[4];
                normals_block(pv, key, n, t, kStreamMove, r, tg.d, bb, q);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = 4 * bb + u;
                    xp[j] = (float)((double)x[j] + eps * q[u]);
                    const double a = (double)x[j] - ref(pv, r, j);
                    const double b = (double)xp[j] - ref(pv, r, j);
                    dle += a * a - b * b;
                }
            }
            ellp = eval<false>(tg, c, pv, r, xp, gp);
            log_alpha = group_sum<LPP>(dle) * c.half_inv_s2r + beta * (ellp - ell);
        } else if constexpr (MOVE == kMala) {
            const double h = 0.5 * eps * eps;
            double dle = 0.0, fwd = 0.0, bwd = 0.0;
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                const double xv = (double)x[j];
                const double ga = -(xv - ref(pv, r, j)) * c.inv_s2r + beta * g[j];
                xp[j] = (float)(xv + h * ga + eps * z[j]);
                const double rr = (double)xp[j] - xv - h * ga;
                fwd = fma(rr, rr, fwd);
            }
            ellp = eval<true, FLAT && !kRoomy>(tg, c, pv, r, xp, gp);
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                const double xv = (double)x[j];
                const double xpv = (double)xp[j];
                const double gap = -(xpv - ref(pv, r, j)) * c.inv_s2r + beta * gp[j];
                const double rr = xv - xpv - h * gap;
                bwd = fma(rr, rr, bwd);
                const double a = xv - ref(pv, r, j);
                const double b = xpv - ref(pv, r, j);
                dle += a * a - b * b;
            }
            const double inv2e2 = 1.0 / (2.0 * eps * eps);
            log_alpha = group_sum<LPP>(dle) * c.half_inv_s2r + beta * (ellp - ell) -
                        group_sum<LPP>(bwd) * inv2e2 + group_sum<LPP>(fwd) * inv2e2;
        } else {
            // HMC: unit mass, L leapfrog steps; positions are stored (rounded) states.
            double mom[DPL];
            double kin0 = 0.0;
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                mom[j] = z[j];
                xp[j] = x[j];
                gp[j] = g[j];
                kin0 += 0.5 * mom[j] * mom[j];
            }
            ellp = ell;
            const double he = 0.5 * eps;
            // the force at the end of a leapfrog step is the next one's at its start
            double force[DPL];
#pragma unroll
            for (int j = 0; j < DPL; ++j)
                force[j] = -((double)xp[j] - ref(pv, r, j)) * c.inv_s2r + beta * gp[j];
            // the first evaluation of a trajectory looks for the components near
            // its particles; the others do where that found few
            if constexpr (!FLAT) {
                bool few = pv.lmf != nullptr;
                for (int l = 0; l < L; ++l) {
#pragma unroll
                    for (int j = 0; j < DPL; ++j) {
                        mom[j] += he * force[j];
                        xp[j] = (float)((double)xp[j] + eps * mom[j]);
                    }
                    ellp = eval<true>(tg, c, pv, r, xp, gp, &few, l + 1 == L);
#pragma unroll
                    for (int j = 0; j < DPL; ++j) {
                        force[j] = -((double)xp[j] - ref(pv, r, j)) * c.inv_s2r + beta * gp[j];
                        mom[j] += he * force[j];
                    }
                }
            } else {
                auto drift = [&] {
#pragma unroll
                    for (int j = 0; j < DPL; ++j) {
                        mom[j] += he * force[j];
                        xp[j] = (float)((double)xp[j] + eps * mom[j]);
                    }
                };
                auto kick = [&] {
#pragma unroll
                    for (int j = 0; j < DPL; ++j) {
                        force[j] = -((double)xp[j] - ref(pv, r, j)) * c.inv_s2r + beta * gp[j];
                        mom[j] += he * force[j];
                    }
                };
                int l = 0;
                bool drifted = false;  // the position of step l is there already
                if constexpr (kLooks) {
                    const bool look = pv.lmf && tg.K > 1 && (!wait || (*wait & 15) == 0);
                    while (look && l < L && !drifted) {
                        drift();
                        const ParView pf = fresh(pv);
                        uint32_t near;
                        if (near_components(tg, pf, r, xp, near)) {
                            ellp = mixture_few<true>(tg, c, pf, r, xp, gp, near, l + 1 == L);
                            kick();
                            ++l;
                        } else {
                            drifted = true;
                        }
                    }
                    if (wait) {
                        if (look)
                            *wait = (drifted && l == 0) ? look_in_vain(*wait) : 0;
                        else if (*wait & 15)
                            --*wait;
                    }
                }
                // ell is wanted at the end only (without registers for a second copy
                // of the evaluation it is formed each time)
                for (; l + (kRoomy ? 1 : 0) < L; ++l) {
                    if (!drifted) drift();
                    drifted = false;
                    ellp = eval<true, true>(tg, c, pv, r, xp, gp, nullptr, !kRoomy);
                    kick();
                }
                if (kRoomy && l < L) {
                    if (!drifted) drift();
                    ellp = eval<true, true>(tg, c, pv, r, xp, gp);
                    kick();
                }
            }
            double kin1 = 0.0, dle = 0.0;
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                kin1 += 0.5 * mom[j] * mom[j];
                const double a = (double)x[j] - ref(pv, r, j);
                const double b = (double)xp[j] - ref(pv, r, j);
                dle += a * a - b * b;
            }
            log_alpha = group_sum<LPP>(dle) * c.half_inv_s2r + beta * (ellp - ell) -
                        group_sum<LPP>(kin1) + group_sum<LPP>(kin0);
        }
        const uint4 w = draw_block(key, n, t, kStreamAccept, 0u, 0u);
        return (forced >= 0) ? (forced != 0) : (-0.5 * minus2_log_word(*pv.nt, w.x) < log_alpha);
    }
};

// ---------------------------------------------------------------------------
// OAIS: persistent tiles, streamed moments.
// ---------------------------------------------------------------------------
constexpr int kTC = 8;      // steps buffered before a transposed reduction
constexpr int kWavesPerBlock = 4;

// Minimum waves per SIMD requested from the compiler for the resampling
// variant's step kernel: four where a lane holds 4 coordinates or a step needs no
// gradients of a mixture, three for HMC with 8 (the d = 100, 8-component
// step at N = 65536: 150 us on two waves, 126 us on three, over 200 on
// four, whose 128-register budget spills inside the trajectory), two for MALA on
// mixtures with 8 (d = 100, 8 components, 40 steps of N = 30000: 2.59 ms, on three
// 2.68), the compiler's choice for wider lanes (which would spill heavily).
template <int FAM, int MOVE, int DPL>
struct MinWaves {
    static constexpr int value = DPL > 8                        ? 1
                                 : DPL <= 4                     ? 4
                                 : MOVE == kHmc                 ? 3
                                 : FAM == kGmm && MOVE == kMala ? 2
                                                                : 4;
};

// The AIS sweeps' slots give the chip at most two waves per SIMD: lanes of up to
// 12 coordinates are kept within the registers of two, wider ones (which would
// spill) are the compiler's choice.
template <int DPL>
struct SweepWaves {
    static constexpr int value = DPL <= 12 ? 2 : 1;
};

// log of w_{t-1} (g_t)^i for a record v = (log w_{t-1}, log g_t): g^0 = 1 also
// where g = 0 (log g = -inf, a zero likelihood), so i = 0 takes log w alone.
__device__ __forceinline__ double mom_term(double2 v, int i)
{
    return (i == 0) ? v.x : v.x + (double)i * v.y;
}

// All tiles of one slot of one problem, in tile order (one wave).  The
// moments of a slot therefore accumulate in the same order whichever wave,
// kernel or launch processes the slot.
template <int FAM, int MOVE, int LPP, int DPL>
__device__ __forceinline__ void oais_slot(const SweepArgs& a, const ParView& pv, const Consts& c,
                                          int64_t slot, double2 (&rec)[kTC][kWave / LPP],
                                          uint32_t (&cntb)[kTC])
{
    constexpr int P = kWave / LPP;
    constexpr int PP = (P + 7) / 8;  // particles per reduction lane
    const int lane = threadIdx.x & (kWave - 1);
    const int r = lane % LPP;
    const int pl = lane / LPP;
    const int T = a.T;
    const int d = a.tg.d;
    const bool grad = uses_grad(MOVE);

    // Fold TC buffered steps of this tile into the slot's accumulators.  For
    // the final entry (fin) the fourth field keeps the largest log w instead
    // of an accepted count.  Bound by VALU issue: the 24 exponentials a lane for 8
    // steps run without branches, and lane part i of a step folds sum i, so that one
    // logarithm and one log_add serve the three (2^22 particles at d = 10,
    // 64 steps: 9.15 -> 8.0 ms).  The functions and
    // their order stay those of one lane after the other: where one particle holds
    // all the weight the discrepancy L_2 - 2 L_1 + L_0 is what their roundings leave.
    auto flush = [&](int64_t slot, bool first, int e0, int cnt, bool fin) {
        wave_sync();
        const int tcl = lane % kTC;
        const int part = lane / kTC;
        // the maximum over the tile's particles first (an xor butterfly over
        // the lanes of one step: every lane ends with the same value), then
        // one exponential per term against it and a butterfly sum: no
        // rescaling exponentials in the merge
        double m[3] = {-INFINITY, -INFINITY, -INFINITY};
        double s[3] = {0.0, 0.0, 0.0};
        if (tcl < cnt) {
#pragma unroll
            for (int q = 0; q < PP; ++q) {
                const int p = part * PP + q;
                if (p < P) {
                    const double2 v = rec[tcl][p];
#pragma unroll
                    for (int i = 0; i < 3; ++i) m[i] = fmax(m[i], mom_term(v, i));
                }
            }
        }
#pragma unroll
        for (int o = kTC; o < kWave; o <<= 1)
#pragma unroll
            for (int i = 0; i < 3; ++i) m[i] = fmax(m[i], __shfl_xor(m[i], o, kWave));
        if (tcl < cnt) {
            // without a finite maximum the terms are -inf and the sum stays 0
            double base[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) base[i] = (m[i] > -INFINITY) ? m[i] : 0.0;
#pragma unroll
            for (int q = 0; q < PP; ++q) {
                const int p = part * PP + q;
                if (p < P) {
                    const double2 v = rec[tcl][p];
#pragma unroll
                    for (int i = 0; i < 3; ++i) s[i] += exp(mom_term(v, i) - base[i]);
                }
            }
        }
#pragma unroll
        for (int o = kTC; o < kWave; o <<= 1)
#pragma unroll
            for (int i = 0; i < 3; ++i) s[i] += __shfl_xor(s[i], o, kWave);
        if (part < 4 && tcl < cnt) {
            double* e = a.part + ((size_t)slot * (T + 1) + (size_t)(e0 + tcl)) * 4 + part;
            const double old = first ? -INFINITY : *e;
            if (part == 3) {
                if (fin)
                    *e = first ? m[0] : fmax(old, m[0]);
                else
                    *e = (first ? 0.0 : old) + (double)cntb[tcl];
            } else {
                // (a sum that is zero or not a number, of a NaN weight, adds nothing)
                const double L = lse_value(part == 0 ? m[0] : (part == 1 ? m[1] : m[2]),
                                           part == 0 ? s[0] : (part == 1 ? s[1] : s[2]));
                *e = first ? L : log_add(old, L);
            }
        }
        wave_sync();
    };

    {
        for (int64_t tile = slot; tile < a.ntiles; tile += a.S) {
            const bool first = (tile == slot);
            const int64_t n64 = tile * P + pl;
            const bool valid = n64 < a.N;
            const uint32_t n = (uint32_t)n64;
            float x[DPL];
            double g[DPL];
            double ell, lw;
            uint32_t accw;
            if (a.sx) {
                // a segment between fixed resampling times: the state the
                // previous segment (or the initial draw) left; lanes past N
                // work on a copy of the last particle and write nothing
                const int64_t nl = valid ? n64 : a.N - 1;
#pragma unroll
                for (int j = 0; j < DPL; ++j) {
                    const int i = r * DPL + j;
                    x[j] = (i < d) ? a.sx[(size_t)nl * d + i] : 0.f;
                    g[j] = (grad && i < d) ? a.sg[(size_t)nl * d + i] : 0.0;
                }
                ell = a.sell[nl];
                lw = a.slw[nl];
                accw = a.saccw[nl];
            } else {
                ell = Particle<FAM, LPP, DPL>::init(a.tg, c, pv, a.key, n, r, x, g, grad);
                lw = 0.0;
                accw = 0;
            }
            int wait = 0;  // see look_in_vain
            const int tb = a.t_begin;
            const int te = a.t_end > 0 ? a.t_end : T;
            for (int t = tb + 1; t <= te; ++t) {
                if (a.ckpt && ((t - 1) % a.ckpt_every) == 0 && valid) {
                    const int nseg = (T + a.ckpt_every - 1) / a.ckpt_every;
                    float* cp = a.ckpt + ((size_t)n64 * nseg + (t - 1) / a.ckpt_every) * d;
#pragma unroll
                    for (int j = 0; j < DPL; ++j) {
                        const int i = r * DPL + j;
                        if (i < d) cp[i] = x[j];
                    }
                }
                const double lg = (a.beta[t] - a.beta[t - 1]) * ell;
                const int tc = (t - tb - 1) % kTC;
                if (r == 0)
                    rec[tc][pl] = valid ? make_double2(lw, lg) : make_double2(-INFINITY, 0.0);
                lw += lg;
                const bool acc = Particle<FAM, LPP, DPL>::template move<MOVE>(
                    a.tg, c, pv, a.key, n, (uint32_t)t, r, a.leapfrog, a.beta[t], a.eps[t - 1], x,
                    ell, g, -1, &wait);
                const uint64_t bal = __ballot(valid && acc && r == 0);
                if (lane == 0) cntb[tc] = (uint32_t)__popcll(bal);
                accw |= (acc ? 1u : 0u) << ((t - 1) & 31);
                if (((t - 1) & 31) == 31 || t == T) {
                    if (a.acc_bits && valid && r == 0)
                        a.acc_bits[(size_t)n64 * a.acc_words + (t - 1) / 32] = accw;
                    accw = 0;
                }
                if (tc == kTC - 1 || t == te) flush(slot, first, t - 1 - tc, tc + 1, false);
            }
            // final weights -> entry T (log-sum-exp and maximum of log w over the tile)
            if (r == 0) rec[0][pl] = valid ? make_double2(lw, 0.0) : make_double2(-INFINITY, 0.0);
            if (lane == 0) cntb[0] = 0u;
            flush(slot, first, T, 1, true);
            if (valid) {
                if (a.sx) {
#pragma unroll
                    for (int j = 0; j < DPL; ++j) {
                        const int i = r * DPL + j;
                        if (i < d) {
                            a.sx[(size_t)n64 * d + i] = x[j];
                            if (grad) a.sg[(size_t)n64 * d + i] = g[j];
                        }
                    }
                    if (r == 0) {
                        a.sell[n64] = ell;
                        a.slw[n64] = lw;
                        a.saccw[n64] = accw;
                    }
                }
                if (a.lw_out && r == 0) a.lw_out[n64] = lw;
                if (a.x_out) {
#pragma unroll
                    for (int j = 0; j < DPL; ++j) {
                        const int i = r * DPL + j;
                        if (i < d) a.x_out[(size_t)n64 * d + i] = x[j];
                    }
                }
            }
        }
    }
}

template <int FAM, int MOVE, int LPP, int DPL>
__global__ void __launch_bounds__(256, (SweepWaves<DPL>::value)) k_oais_valu(SweepArgs a)
{
    __shared__ double2 sh_rec[kWavesPerBlock][kTC][kWave / LPP];
    __shared__ uint32_t sh_cnt[kWavesPerBlock][kTC];
    extern __shared__ __align__(16) char sh_dyn[];
    __shared__ NormalTables sh_nt;
    const ParView pv = stage_params_lanes<MOVE, LPP, DPL>(a.tg, sh_dyn, &sh_nt);
    const Consts c = make_consts(a.tg);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // wave-uniform
    const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + wv;
    const int64_t W = (int64_t)gridDim.x * kWavesPerBlock;
    for (int64_t slot = gw; slot < a.S; slot += W)
        oais_slot<FAM, MOVE, LPP, DPL>(a, pv, c, slot, sh_rec[wv], sh_cnt[wv]);
}

// Many problems of one (family, move, shape) class in one launch: each wave
// walks the work list of (problem, slot) items; target parameters are read
// from global memory through per-problem views.
template <int FAM, int MOVE, int LPP, int DPL>
__global__ void __launch_bounds__(256, (SweepWaves<DPL>::value)) k_oais_valu_batch(const SweepArgs* __restrict__ args,
                                                         const ParView* __restrict__ views,
                                                         const int2* __restrict__ items,
                                                         int64_t nitems, uint32_t* next)
{
    __shared__ double2 sh_rec[kWavesPerBlock][kTC][kWave / LPP];
    __shared__ uint32_t sh_cnt[kWavesPerBlock][kTC];
    __shared__ NormalTables sh_nt;
    stage_tables(sh_nt);
    __syncthreads();
    // the wave index through readfirstlane, so that the compiler sees the
    // work item, its arguments and its parameter view as wave-uniform (scalar
    // loads into scalar registers instead of per-lane copies in vector
    // registers)
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + wv;
    const int64_t W = (int64_t)gridDim.x * kWavesPerBlock;
    // each wave claims its next item from the work counter (zero at the
    // launch; items longest first: a greedy balance), or without one takes
    // the static round robin; the claim is read back wave-uniform
    auto claim = [&](int64_t prev) -> int64_t {
        if (next == nullptr) return prev < 0 ? gw : prev + W;
        uint32_t v = 0u;
        if ((threadIdx.x & (kWave - 1)) == 0) v = atomicAdd(next, 1u);
        return (int64_t)__builtin_amdgcn_readfirstlane(v);
    };
    for (int64_t it = claim(-1); it < nitems; it = claim(it)) {
        const int2 item = items[it];
        const SweepArgs a = args[item.x];
        ParView pv = views[item.x];
        pv.nt = &sh_nt;
        const Consts c = make_consts(a.tg);
        oais_slot<FAM, MOVE, LPP, DPL>(a, pv, c, (int64_t)item.y, sh_rec[wv], sh_cnt[wv]);
    }
}

// ---------------------------------------------------------------------------
// Adaptive-resampling variant: one launch per step.
// ---------------------------------------------------------------------------
template <int FAM, int MOVE, int LPP, int DPL>
__global__ void __launch_bounds__(256) k_asmc_init(SweepArgs a, AsmcState z)
{
    constexpr int P = kWave / LPP;
    extern __shared__ __align__(16) char sh_dyn[];
    __shared__ NormalTables sh_nt;
    const ParView pv = stage_params_lanes<MOVE, LPP, DPL>(a.tg, sh_dyn, &sh_nt);
    const Consts c = make_consts(a.tg);
    const int lane = threadIdx.x & (kWave - 1);
    const int r = lane % LPP, pl = lane / LPP;
    const int64_t tile =
        (int64_t)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t n64 = tile * P + pl;
    if (tile >= a.ntiles || n64 >= a.N) return;
    if (lane == 0) z.tile_part[(size_t)tile * 8 + 6] = 0.0;
    float x[DPL];
    double g[DPL];
    const double ell = Particle<FAM, LPP, DPL>::init(a.tg, c, pv, a.key, (uint32_t)n64, r, x, g,
                                                     uses_grad(MOVE));
#pragma unroll
    for (int j = 0; j < DPL; ++j) {
        const int i = r * DPL + j;
        if (i < a.tg.d) {
            z.X[(size_t)n64 * a.tg.d + i] = x[j];
            if (uses_grad(MOVE)) z.G[(size_t)n64 * a.tg.d + i] = g[j];
        }
    }
    if (r == 0) {
        z.ell[n64] = ell;
        z.lw[n64] = 0.0;
        z.accw[n64] = 0u;
    }
}

// A lane's coordinates r DPL .. of particle row `row` of an [N][d] array, zero
// beyond d: in quads where d is a multiple of four (rows then start on 16 bytes and
// a quad lies within d or beyond it), one by one otherwise.
template <int DPL>
__device__ __forceinline__ void load_row(const float* __restrict__ p, int64_t row, int d, int r,
                                         float (&x)[DPL])
{
    const float* q = p + (size_t)row * d + r * DPL;
    if (d % 4 == 0) {
#pragma unroll
        for (int j = 0; j < DPL; j += 4) {
            const float4 v = (r * DPL + j < d) ? *reinterpret_cast<const float4*>(q + j)
                                               : make_float4(0.f, 0.f, 0.f, 0.f);
            x[j] = v.x;
            x[j + 1] = v.y;
            x[j + 2] = v.z;
            x[j + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < DPL; ++j) x[j] = (r * DPL + j < d) ? q[j] : 0.f;
    }
}
template <int DPL>
__device__ __forceinline__ void load_row(const double* __restrict__ p, int64_t row, int d, int r,
                                         double (&x)[DPL])
{
    const double* q = p + (size_t)row * d + r * DPL;
    if (d % 4 == 0) {
#pragma unroll
        for (int j = 0; j < DPL; j += 2) {
            const double2 v = (r * DPL + j < d) ? *reinterpret_cast<const double2*>(q + j)
                                                : make_double2(0.0, 0.0);
            x[j] = v.x;
            x[j + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < DPL; ++j) x[j] = (r * DPL + j < d) ? q[j] : 0.0;
    }
}
template <int DPL>
__device__ __forceinline__ void store_row(float* __restrict__ p, int64_t row, int d, int r,
                                          const float (&x)[DPL])
{
    float* q = p + (size_t)row * d + r * DPL;
    if (d % 4 == 0) {
#pragma unroll
        for (int j = 0; j < DPL; j += 4)
            if (r * DPL + j < d)
                *reinterpret_cast<float4*>(q + j) = make_float4(x[j], x[j + 1], x[j + 2], x[j + 3]);
    } else {
#pragma unroll
        for (int j = 0; j < DPL; ++j)
            if (r * DPL + j < d) q[j] = x[j];
    }
}
template <int DPL>
__device__ __forceinline__ void store_row(double* __restrict__ p, int64_t row, int d, int r,
                                          const double (&x)[DPL])
{
    double* q = p + (size_t)row * d + r * DPL;
    if (d % 4 == 0) {
#pragma unroll
        for (int j = 0; j < DPL; j += 2)
            if (r * DPL + j < d) *reinterpret_cast<double2*>(q + j) = make_double2(x[j], x[j + 1]);
    } else {
#pragma unroll
        for (int j = 0; j < DPL; ++j)
            if (r * DPL + j < d) q[j] = x[j];
    }
}

// The launch has at most as many blocks as are resident, and each walks over
// tiles: the staging of the target's parameters and tables (a few us of dependent
// loads) is paid once a block and not once a tile (the d = 100, 8-component HMC step
// of 65536 particles: 195 -> 142 us).
template <int FAM, int MOVE, int LPP, int DPL>
__global__ void __launch_bounds__(256, (MinWaves<FAM, MOVE, DPL>::value))
    k_asmc_step(SweepArgs a, AsmcState z, int t)
{
    if (a.t_stop && t > *a.t_stop) return;  // an online schedule already reached beta = 1
    constexpr int P = kWave / LPP;
    extern __shared__ __align__(16) char sh_dyn[];
    __shared__ NormalTables sh_nt;
    const ParView pv = stage_params_lanes<MOVE, LPP, DPL>(a.tg, sh_dyn, &sh_nt);
    const Consts c = make_consts(a.tg);
    const int lane = threadIdx.x & (kWave - 1);
    const int r = lane % LPP, pl = lane / LPP;
    const int d = a.tg.d;
    const double beta = a.beta[t], dbeta = beta - a.beta[t - 1], eps = a.eps[t - 1];
    // state, ell and (MALA, HMC) grad ell as the previous step left them:
    // after a resampling event at the previous step (its flag is still set:
    // the merge of this step has not run) the gathered copies X2, G2, ell2
    // with log w = 0; this step writes X, G, ell as always, so the gathered
    // state is never copied back (runs without a gather target never resample)
    const bool rs = z.X2 != nullptr && z.scal[2] != 0.0;
    const float* Xs = rs ? z.X2 : z.X;
    const double* Gs = rs ? z.G2 : z.G;
    const double* es = rs ? z.ell2 : z.ell;
    for (int64_t tile = (int64_t)blockIdx.x * kWavesPerBlock +
                        __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
         tile < a.ntiles; tile += (int64_t)gridDim.x * kWavesPerBlock) {
        const int64_t n64 = tile * P + pl;
        const bool valid = n64 < a.N;
        const int64_t nl = valid ? n64 : a.N - 1;  // invalid lanes work on a copy, write nothing
        float x[DPL];
        double g[DPL];
        load_row<DPL>(Xs, nl, d, r, x);
        if constexpr (uses_grad(MOVE)) {
            load_row<DPL>(Gs, nl, d, r, g);
        } else {
#pragma unroll
            for (int j = 0; j < DPL; ++j) g[j] = 0.0;
        }
        double ell = es[nl];
        double lw = rs ? 0.0 : z.lw[nl];
        const double lg = dbeta * ell;
        // tile statistics: lse of lw, lw+lg, lw+2lg, 2(lw+lg) over the tile's
        // particles: the maximum by an xor butterfly over the particle groups
        // (every lane ends with the same value), then the exponentials against
        // it and a butterfly sum.  Where a particle spans four lanes or more, its
        // lane i mod 4 forms statistic i (a quarter of the instructions).
        constexpr int NS = LPP >= 4 ? 1 : 4;
        double m[NS], s[NS];
        {
            const double v4[4] = {lw, lw + lg, lw + 2.0 * lg, 2.0 * (lw + lg)};
            double v[NS];
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                if constexpr (NS == 4)
                    v[i] = v4[i];
                else
                    v[i] = (r & 2) ? ((r & 1) ? v4[3] : v4[2]) : ((r & 1) ? v4[1] : v4[0]);
                m[i] = valid ? v[i] : -INFINITY;
            }
#pragma unroll
            for (int o = LPP; o < kWave; o <<= 1)
#pragma unroll
                for (int i = 0; i < NS; ++i) m[i] = fmax(m[i], __shfl_xor(m[i], o, kWave));
#pragma unroll
            for (int i = 0; i < NS; ++i)
                s[i] = (valid && m[i] > -INFINITY) ? exp(v[i] - m[i]) : 0.0;
#pragma unroll
            for (int o = LPP; o < kWave; o <<= 1)
#pragma unroll
                for (int i = 0; i < NS; ++i) s[i] += __shfl_xor(s[i], o, kWave);
        }
        lw += lg;
        if (lane < 4) {
            // lane i records statistic i
            double mi = m[0], si = s[0];
            if constexpr (NS == 4) {
                mi = (lane & 2) ? ((lane & 1) ? m[3] : m[2]) : ((lane & 1) ? m[1] : m[0]);
                si = (lane & 2) ? ((lane & 1) ? s[3] : s[2]) : ((lane & 1) ? s[1] : s[0]);
            }
            double* tp = z.tile_part + (size_t)tile * 8;
            tp[lane] = lse_value(mi, si);
            if (lane == 1) tp[4] = mi;  // max of log w_{t^-}
        }
        bool acc;
        if constexpr (uses_grad(MOVE)) {
            // a rejected proposal's state is still in memory: neither it nor its
            // gradient is held over the step, and it is written only where it
            // comes from the gathered copies
            constexpr bool kFlat = MOVE == kHmc && DPL > 8;
            constexpr bool kWaits = kFlat && Particle<FAM, LPP, DPL>::kLooks;
            int wait = 0;  // kept with the tile from step to step
            if constexpr (kWaits)
                wait = __builtin_amdgcn_readfirstlane((int)z.tile_part[(size_t)tile * 8 + 6]);
            float xp[DPL];
            double gp[DPL], ellp;
            acc = Particle<FAM, LPP, DPL>::template propose<MOVE, kFlat>(a.tg, c, pv, a.key, (uint32_t)nl,
                                                                  (uint32_t)t, r, a.leapfrog, beta, eps,
                                                                  x, ell, g, xp, ellp, gp, -1, &wait);
            if constexpr (kWaits)
                if (lane == 0) z.tile_part[(size_t)tile * 8 + 6] = (double)wait;
            if (acc) ell = ellp;
            if (rs && !acc) {
                load_row<DPL>(Xs, nl, d, r, xp);
                load_row<DPL>(Gs, nl, d, r, gp);
            }
            if (valid && (rs || acc)) {
                store_row<DPL>(z.X, n64, d, r, xp);
                store_row<DPL>(z.G, n64, d, r, gp);
            }
        } else {
            acc = Particle<FAM, LPP, DPL>::template move<MOVE>(a.tg, c, pv, a.key, (uint32_t)nl,
                                                               (uint32_t)t, r, a.leapfrog, beta, eps, x,
                                                               ell, g);
            if (valid && (rs || acc)) store_row<DPL>(z.X, n64, d, r, x);
        }
        const uint64_t bal = __ballot(valid && acc && r == 0);
        if (lane == 0) z.tile_part[(size_t)tile * 8 + 5] = (double)__popcll(bal);
        if (valid) {
            if (r == 0) {
                z.ell[n64] = ell;
                z.lw[n64] = lw;
                uint32_t w = z.accw[n64] | ((acc ? 1u : 0u) << ((t - 1) & 31));
                if (((t - 1) & 31) == 31 || t == a.T) {
                    if (a.acc_bits) a.acc_bits[(size_t)n64 * a.acc_words + (t - 1) / 32] = w;
                    w = 0u;
                }
                z.accw[n64] = w;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Final-iteration rejuvenation (Sec. "Computing expectations"): after the
// last annealing step the population is resampled and N chains run T steps of
// the forward kernel at beta = 1 (step size eps_T), chain n from particle
// anc[n]; its states feed the expectations.  One wave per tile as in the
// sweep; the chain draws with counters (n, T + s), s = 1..T.  Sums of x_i and
// x_i^2 over the chain are kept per lane (in step order), summed over the
// wave's particles by an xor butterfly and written per tile.
// ---------------------------------------------------------------------------
template <int FAM, int MOVE, int LPP, int DPL>
__global__ void __launch_bounds__(256) k_rejuv(RejuvArgs R)
{
    constexpr int P = kWave / LPP;
    extern __shared__ __align__(16) char sh_dyn[];
    const SweepArgs& a = R.a;
    __shared__ NormalTables sh_nt;
    const ParView pv = stage_params_lanes<MOVE, LPP, DPL>(a.tg, sh_dyn, &sh_nt);
    const Consts c = make_consts(a.tg);
    const int lane = threadIdx.x & (kWave - 1);
    const int r = lane % LPP, pl = lane / LPP;
    const int64_t tile =
        (int64_t)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (tile >= a.ntiles) return;  // whole wave leaves together
    const int64_t n64 = tile * P + pl;
    const bool valid = n64 < a.N;
    const int d = a.tg.d;
    // the host checked the event, so every ancestor is a particle index
    const int64_t src = R.anc[valid ? n64 : a.N - 1];
    float x[DPL];
    double g[DPL];
#pragma unroll
    for (int j = 0; j < DPL; ++j) {
        const int i = r * DPL + j;
        x[j] = (i < d) ? R.x_in[(size_t)src * d + i] : 0.f;
        g[j] = 0.0;
    }
    double ell = uses_grad(MOVE) ? Particle<FAM, LPP, DPL>::template eval<true>(a.tg, c, pv, r, x, g)
                                 : Particle<FAM, LPP, DPL>::template eval<false>(a.tg, c, pv, r, x, g);
    double s1[DPL], s2[DPL];
#pragma unroll
    for (int j = 0; j < DPL; ++j) s1[j] = s2[j] = 0.0;
    uint32_t na = 0;
    int wait = 0;
    for (int s = 1; s <= a.T; ++s) {
        const bool acc = Particle<FAM, LPP, DPL>::template move<MOVE>(
            a.tg, c, pv, a.key, (uint32_t)n64, (uint32_t)(a.T + s), r, a.leapfrog, 1.0, R.eps, x,
            ell, g, -1, &wait);
        na += acc ? 1u : 0u;
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            const double v = (double)x[j];
            s1[j] += v;
            s2[j] += v * v;
        }
    }
    if (valid && R.x_out) {
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            const int i = r * DPL + j;
            if (i < d) R.x_out[(size_t)n64 * d + i] = x[j];
        }
    }
    // sums over the wave's particles (lanes r, r + LPP, ... hold the same coordinates)
    double cnt = (valid && r == 0) ? (double)na : 0.0;
#pragma unroll
    for (int j = 0; j < DPL; ++j) {
        if (!valid) s1[j] = s2[j] = 0.0;
#pragma unroll
        for (int o = LPP; o < kWave; o <<= 1) {
            s1[j] += __shfl_xor(s1[j], o, kWave);
            s2[j] += __shfl_xor(s2[j], o, kWave);
        }
    }
    cnt = wave_sum(cnt);
    double* out = R.tsum + (size_t)tile * (2 * d + 1);
    if (pl == 0) {
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            const int i = r * DPL + j;
            if (i < d) {
                out[i] = s1[j];
                out[d + i] = s2[j];
            }
        }
        if (r == 0) out[2 * d] = cnt;
    }
}

// ---------------------------------------------------------------------------
// Parallel tempering (Sec. "Computational duality with parallel tempering"):
// one workgroup per PT copy, replica r of the copy on particle slot r of the
// workgroup (LPP lanes), at temperature tau[r].  Iteration t: every replica
// takes one step of the forward kernel at its temperature (counters (replica,
// t)); then one thread per proposed pair (n, n + 1) of the parity of t decides
// the swap of temperatures (stream 4, counter (copy (N' + 1) + n, t)); then
// the stepping-stone terms (one thread per temperature, a running maximum and
// scaled sum), round trips (one thread per replica) and the target chain's
// sums (the replica at N') are taken.  Swaps exchange temperatures, not states.
// ---------------------------------------------------------------------------
constexpr uint32_t kStreamSwap = 4;

// At most 8 waves per copy (512 threads): two waves per SIMD leave the move
// arithmetic its registers (at 1024 threads the compiler caps a lane at 128
// registers and spills several hundred bytes per lane).
constexpr int kPtMaxThreads = 512;

template <int FAM, int MOVE, int LPP, int DPL>
__global__ void __launch_bounds__(kPtMaxThreads) k_pt(PtArgs A)
{
    constexpr int P = kWave / LPP;
    extern __shared__ __align__(16) char sh_dyn[];
    const SweepArgs& a = A.a;
    __shared__ NormalTables sh_nt;
    const ParView pv = stage_params_lanes<MOVE, LPP, DPL>(a.tg, sh_dyn, &sh_nt);
    const Consts c = make_consts(a.tg);
    const int R = A.Np + 1;
    const int Np = A.Np;
    size_t off = (params_bytes_lanes(a.tg, MOVE, LPP, DPL) + 15) & ~(size_t)15;
    double* Lsh = reinterpret_cast<double*>(sh_dyn + off);   // [R] ell of replica r
    double* rsum = Lsh + R;                                   // [Np] summed rejections
    int* tau = reinterpret_cast<int*>(rsum + Np);             // [R] temperature of replica r
    int* rep = tau + R;                                       // [R] replica at temperature n
    int* side = rep + R;                                      // [R] round-trip state
    double* red = reinterpret_cast<double*>(side + R + ((R & 1) ? 1 : 0));  // [16]
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = tid / kWave;
    const int r = lane % LPP;
    const int slot = wv * P + lane / LPP;   // replica of this lane group
    const bool live = slot < R;
    const int k = blockIdx.x;
    const uint32_t gid = (uint32_t)(k * R + (live ? slot : 0));
    const int d = a.tg.d;
    for (int i = tid; i < R; i += blockDim.x) {
        tau[i] = i;
        rep[i] = i;
        side[i] = (i == 0) ? 0 : -1;
    }
    for (int i = tid; i < Np; i += blockDim.x) rsum[i] = 0.0;
    float x[DPL];
    double g[DPL];
    double ell = Particle<FAM, LPP, DPL>::init(a.tg, c, pv, a.key, gid, r, x, g, uses_grad(MOVE));
    double f1[DPL], f2[DPL];
#pragma unroll
    for (int j = 0; j < DPL; ++j) f1[j] = f2[j] = 0.0;
    double sm = -INFINITY, ss = 0.0;  // stepping stone of temperature tid (tid < Np)
    double trips = 0.0;               // round trips of replica tid (tid < R)
    int wait = 0;
    __syncthreads();
    for (int t = 1; t <= a.T; ++t) {
        const int n = live ? tau[slot] : 0;
        Particle<FAM, LPP, DPL>::template move<MOVE>(a.tg, c, pv, a.key, gid, (uint32_t)t, r,
                                                     a.leapfrog, A.beta[n], A.eps[n], x, ell, g, -1,
                                                     &wait);
        if (live && r == 0) Lsh[slot] = ell;
        __syncthreads();
        // swaps of the pairs (n, n + 1), n of the parity of t
        {
            const int np = ((t & 1) ? 1 : 0) + 2 * tid;
            if (np + 1 < R) {
                const int ra = rep[np], rb = rep[np + 1];
                const double la = (A.beta[np + 1] - A.beta[np]) * (Lsh[ra] - Lsh[rb]);
                const uint4 w = draw_block(a.key, (uint32_t)(k * R + np), (uint32_t)t, kStreamSwap,
                                           0u, 0u);
                const double acc = (la >= 0.0) ? 1.0 : ((la == la) ? exp(la) : 0.0);
                rsum[np] += 1.0 - acc;
                if (-0.5 * minus2_log_word(*pv.nt, w.x) < la) {
                    rep[np] = rb;
                    rep[np + 1] = ra;
                    tau[ra] = np + 1;
                    tau[rb] = np;
                }
            }
        }
        __syncthreads();
        if (tid < R) {
            const int tr = tau[tid];
            if (tr == Np && side[tid] == 0) side[tid] = 1;
            if (tr == 0) {
                if (side[tid] == 1) trips += 1.0;
                side[tid] = 0;
            }
        }
        if (tid < Np) {
            const double v = (A.beta[tid + 1] - A.beta[tid]) * Lsh[rep[tid]];
            if (v > -INFINITY) {
                const bool up = v > sm;
                const double e = exp(up ? sm - v : v - sm);
                ss = up ? ss * e + 1.0 : ss + e;
                sm = up ? v : sm;
            }
        }
        if (live && tau[slot] == Np) {
#pragma unroll
            for (int j = 0; j < DPL; ++j) {
                const double v = (double)x[j];
                f1[j] += v;
                f2[j] += v * v;
            }
        }
        __syncthreads();
    }
    // per-copy outputs: stepping stone (max, scaled sum), rejections, round
    // trips, target-chain sums over the copy's replicas (fixed order)
    double* o = A.out + (size_t)k * A.stride;
    if (tid < Np) {
        o[2 * tid] = sm;
        o[2 * tid + 1] = ss;
        o[2 * Np + tid] = rsum[tid];
    }
    double tr = wave_sum(trips);
    if (lane == 0) red[wv] = tr;
#pragma unroll
    for (int j = 0; j < DPL; ++j) {
        if (!live) f1[j] = f2[j] = 0.0;
#pragma unroll
        for (int q = LPP; q < kWave; q <<= 1) {
            f1[j] += __shfl_xor(f1[j], q, kWave);
            f2[j] += __shfl_xor(f2[j], q, kWave);
        }
    }
    double* fo = A.fpart + ((size_t)k * 16 + wv) * 2 * d;
    if (lane < LPP) {
#pragma unroll
        for (int j = 0; j < DPL; ++j) {
            const int i = r * DPL + j;
            if (i < d) {
                fo[i] = f1[j];
                fo[d + i] = f2[j];
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int i = 0; i < (int)(blockDim.x / kWave); ++i) s += red[i];
        o[3 * Np] = s;
        o[3 * Np + 1] = (double)(blockDim.x / kWave);
    }
}

// ell and grad ell at given binary32 states: the particle's coordinates are
// loaded into the lane layout (zero beyond d) and evaluated by the sweep's
// Particle::eval, one lane group per particle.
template <int FAM, int LPP, int DPL>
__global__ void __launch_bounds__(256) k_target_eval(EvalArgs E)
{
    constexpr int P = kWave / LPP;
    extern __shared__ __align__(16) char sh_dyn[];
    const SweepArgs& a = E.a;
    const ParView pv = stage_params_lanes<kMala, LPP, DPL>(a.tg, sh_dyn, nullptr);
    const Consts c = make_consts(a.tg);
    const int lane = threadIdx.x & (kWave - 1);
    const int r = lane % LPP, pl = lane / LPP;
    const int64_t tile =
        (int64_t)blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (tile >= a.ntiles) return;
    // a tile's particles beyond N evaluate zeros and write nothing, so the
    // lane groups of a wave stay converged through the evaluation
    const int64_t n64 = tile * P + pl;
    const bool valid = n64 < a.N;
    const int d = a.tg.d;
    float x[DPL];
    double g[DPL];
#pragma unroll
    for (int j = 0; j < DPL; ++j) {
        const int i = r * DPL + j;
        x[j] = (valid && i < d) ? E.x[(size_t)n64 * d + i] : 0.f;
    }
    const double ell = Particle<FAM, LPP, DPL>::template eval<true>(a.tg, c, pv, r, x, g);
    if (!valid) return;
#pragma unroll
    for (int j = 0; j < DPL; ++j) {
        const int i = r * DPL + j;
        if (i < d) E.grad[(size_t)n64 * d + i] = g[j];
    }
    if (r == 0) E.ell[n64] = ell;
}

static_assert(sizeof(NormalTables) == kNormalTableBytes, "counted beside the dynamic LDS");

template <int FAM, int MOVE, int LPP, int DPL>
struct Launch {
    static hipError_t oais(const SweepArgs& a, int grid_waves, hipStream_t st)
    {
        const int blocks = (grid_waves + kWavesPerBlock - 1) / kWavesPerBlock;
        hipLaunchKernelGGL((k_oais_valu<FAM, MOVE, LPP, DPL>), dim3(blocks), dim3(256),
                           params_bytes_lanes(a.tg, MOVE, LPP, DPL), st, a);
        return hipGetLastError();
    }
    static hipError_t batch(const SweepArgs* args, const ParView* views, const int2* items,
                            int64_t nitems, uint32_t* next, int grid_waves, hipStream_t st)
    {
        const int blocks = (grid_waves + kWavesPerBlock - 1) / kWavesPerBlock;
        hipLaunchKernelGGL((k_oais_valu_batch<FAM, MOVE, LPP, DPL>), dim3(blocks), dim3(256), 0, st,
                           args, views, items, nitems, next);
        return hipGetLastError();
    }
    static hipError_t init(const SweepArgs& a, const AsmcState& z, hipStream_t st)
    {
        const int64_t blocks = (a.ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
        hipLaunchKernelGGL((k_asmc_init<FAM, MOVE, LPP, DPL>), dim3((unsigned)blocks), dim3(256),
                           params_bytes_lanes(a.tg, MOVE, LPP, DPL), st, a, z);
        return hipGetLastError();
    }
    static hipError_t rejuv(const RejuvArgs& R, hipStream_t st)
    {
        const int64_t blocks = (R.a.ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
        hipLaunchKernelGGL((k_rejuv<FAM, MOVE, LPP, DPL>), dim3((unsigned)blocks), dim3(256),
                           params_bytes_lanes(R.a.tg, MOVE, LPP, DPL), st, R);
        return hipGetLastError();
    }
    static hipError_t pt(const PtArgs& A, hipStream_t st)
    {
        constexpr int P = kWave / LPP;
        const int waves = (A.Np + 1 + P - 1) / P;
        const size_t shb = pt_shared_bytes(A, LPP, DPL);
        hipLaunchKernelGGL((k_pt<FAM, MOVE, LPP, DPL>), dim3((unsigned)A.K), dim3(waves * kWave),
                           shb, st, A);
        return hipGetLastError();
    }
    static hipError_t eval(const EvalArgs& E, hipStream_t st)
    {
        // one instantiation per family: the evaluation does not depend on the move
        if constexpr (MOVE == kMala || (FAM == kUnid && MOVE == kRwmh)) {
            const int64_t blocks = (E.a.ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
            hipLaunchKernelGGL((k_target_eval<FAM, LPP, DPL>), dim3((unsigned)blocks), dim3(256),
                               params_bytes_lanes(E.a.tg, kMala, LPP, DPL), st, E);
            return hipGetLastError();
        } else {
            (void)E;
            (void)st;
            return hipErrorInvalidValue;
        }
    }
    static hipError_t step(const SweepArgs& a, const AsmcState& z, int t, hipStream_t st)
    {
        // resident blocks: as many as the registers of this instantiation and its LDS allow
        static const int by_registers = [] {
            int n = 0;
            const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &n, reinterpret_cast<const void*>(&k_asmc_step<FAM, MOVE, LPP, DPL>), 256, 0);
            return (e == hipSuccess && n > 0) ? n : 2;
        }();
        const size_t lds = params_bytes_lanes(a.tg, MOVE, LPP, DPL);
        const int per_cu = std::min<int>(by_registers, (int)(kLdsPerCu / (lds + sizeof(NormalTables))));
        const int64_t blocks = std::min<int64_t>((a.ntiles + kWavesPerBlock - 1) / kWavesPerBlock,
                                                 (int64_t)kFillCus * per_cu);
        hipLaunchKernelGGL((k_asmc_step<FAM, MOVE, LPP, DPL>), dim3((unsigned)blocks), dim3(256),
                           lds, st, a, z, t);
        return hipGetLastError();
    }
};

template <int FAM, int MOVE>
hipError_t valu_dispatch(int what, const SweepArgs& a, const ValuShape& s, int gw,
                           const AsmcState* z, int t, hipStream_t st, const ValuBatch* b,
                           const void* ext)
{
    const RejuvArgs* rj = static_cast<const RejuvArgs*>(ext);
    const PtArgs* pt = static_cast<const PtArgs*>(ext);
    const EvalArgs* ev = static_cast<const EvalArgs*>(ext);
#define OASMC_CASE(L, D)                                                     \
    if (s.lpp == L && s.dpl == D) {                                          \
        if (what == 0) return Launch<FAM, MOVE, L, D>::oais(a, gw, st);      \
        if (what == 1) return Launch<FAM, MOVE, L, D>::init(a, *z, st);      \
        if (what == 3)                                                       \
            return Launch<FAM, MOVE, L, D>::batch(b->args, b->views, b->items, \
                                                  b->nitems, b->next, gw, st); \
        if (what == 4) return Launch<FAM, MOVE, L, D>::rejuv(*rj, st);       \
        if (what == 5) return Launch<FAM, MOVE, L, D>::pt(*pt, st);          \
        if (what == 6) return Launch<FAM, MOVE, L, D>::eval(*ev, st);        \
        return Launch<FAM, MOVE, L, D>::step(a, *z, t, st);                  \
    }
    OASMC_CASE(1, 4)
    if constexpr (FAM == kUnid) return hipErrorInvalidValue;  // d = 2: one lane of 4 only
    OASMC_CASE(1, 8)
    OASMC_CASE(1, 12)
    OASMC_CASE(1, 16)
    OASMC_CASE(1, 20)
    OASMC_CASE(1, 24)
    OASMC_CASE(2, 16)
    OASMC_CASE(4, 16)
    OASMC_CASE(8, 16)
    OASMC_CASE(16, 16)
    OASMC_CASE(8, 8)
    OASMC_CASE(16, 8)
    OASMC_CASE(4, 8)
    OASMC_CASE(8, 4)
#undef OASMC_CASE
    return hipErrorInvalidValue;
}

}  // namespace oasmc
