// sweep_common.hip -- the kernels shared by every annealing pass: the
// slot-order merge of streamed moments, the per-step merge and trigger of the
// resampling variant, the integer-CDF systematic resampler, raw Philox blocks,
// and the host-side dispatch to the per-(family, move) sweep instantiations.
#include "kernels.hpp"

namespace oasmc {

// Merge the S slot partials of one entry (one workgroup per entry): the
// log-sum-exps are a maximum and then a sum of exp(x - max) in a fixed order,
// that of one wave whose lanes take slots lane, lane + 64, ... (deterministic, and
// independent of the grid): log_g[i*T + e] for e < T, the accept fraction, and
// log Z_hat from entry T.  Bound by latency (a cache line a slot, few entries) and
// the exponentials: the waves take groups of 64 slots in turn, and waves 0 to 2 add
// one of the three columns each from LDS, group after group, in the order of the
// slots (20011 HMC particles in segments: 37 -> 12 us a merge).
constexpr int kEntryWaves = 8;
constexpr int kEntryThreads = kEntryWaves * kWave;

struct EntryShared {
    double red[kEntryWaves][4];
    double term[2][kEntryWaves][3][kWave];
    double L[3];
};

__device__ __forceinline__ void merge_entry(EntryShared& sh, const double* __restrict__ part, int64_t S,
                                            int T, int e, double (&L)[3], double& cnt)
{
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const double* col = part + (size_t)e * 4;
    const size_t row = (size_t)(T + 1) * 4;
    double m[3] = {-INFINITY, -INFINITY, -INFINITY};
    double c = 0.0;
    for (int64_t s = tid; s < S; s += kEntryThreads) {
        const double* p = col + (size_t)s * row;
#pragma unroll
        for (int i = 0; i < 3; ++i) m[i] = fmax(m[i], p[i]);
        c += p[3];  // counts: whole numbers, the same in any order
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) m[i] = wave_max(m[i]);
    c = wave_sum(c);
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) sh.red[w][i] = m[i];
        sh.red[w][3] = c;
    }
    __syncthreads();
    cnt = 0.0;
#pragma unroll
    for (int u = 0; u < kEntryWaves; ++u) {
#pragma unroll
        for (int i = 0; i < 3; ++i) m[i] = fmax(m[i], sh.red[u][i]);
        cnt += sh.red[u][3];
    }
    double sum = 0.0;
    int buf = 0;
    for (int64_t s0 = 0; s0 < S; s0 += kEntryThreads, buf ^= 1) {
        const int64_t s = s0 + tid;
        const double* p = col + (size_t)(s < S ? s : S - 1) * row;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            sh.term[buf][w][i][lane] =
                (s < S && m[i] > -INFINITY && p[i] > -INFINITY) ? exp(p[i] - m[i]) : 0.0;
        __syncthreads();
        if (w < 3) {
#pragma unroll
            for (int u = 0; u < kEntryWaves; ++u) sum += sh.term[buf][u][w][lane];
        }
    }
    if (w < 3) {
        const double l = lse_value(w == 0 ? m[0] : (w == 1 ? m[1] : m[2]), wave_sum(sum));
        if (lane == 0) sh.L[w] = l;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 3; ++i) L[i] = sh.L[i];
}

__global__ void __launch_bounds__(kEntryThreads) k_merge_slots(const double* __restrict__ part, int64_t S,
                                                       int T, int64_t N, double* log_g, double* acc,
                                                       double* logZ)
{
    const int e = blockIdx.x;
    double L[3], cnt;
    __shared__ EntryShared sh;
    merge_entry(sh, part, S, T, e, L, cnt);
    if (threadIdx.x != 0) return;
    if (e < T) {
#pragma unroll
        for (int i = 0; i < 3; ++i) log_g[(size_t)i * T + e] = L[i];
        acc[e] = cnt / (double)N;
    } else {
        logZ[0] = L[0] - log((double)N);
    }
}

// The per-step merge of the resampling variant, in two levels with a fixed
// order (deterministic, independent of timing): block b of the first level
// reduces a contiguous range of tile records to one record (log-sum-exps as a
// maximum and then a sum of exp(x - max)); the last block to finish then
// merges the block records, records the moments, ESS and CESS, decides the
// event and adds the log Z_hat increment (one launch).
constexpr int kMergeThreads = 256;

__device__ __forceinline__ int merge_blocks(int64_t ntiles)
{
    const int64_t nb = (ntiles + kMergeThreads - 1) / kMergeThreads;
    return (int)(nb < kAsmcMergeBlocks ? nb : kAsmcMergeBlocks);
}

// Second level, by the four waves of a block: wave i forms log-sum-exp i of the block
// records; then one thread the moments, ESS and CESS, the event decision and the
// log Z_hat increment.
__device__ __forceinline__ void asmc_merge_final(const SweepArgs& a, const AsmcState& z, int t,
                                                 int trigger, double nu, double (&shl)[4])
{
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int nb = merge_blocks(a.ntiles);
    const double* rec = z.blk_part + (size_t)lane * 8;
    const bool have = lane < nb;
    const double v = have ? rec[w] : -INFINITY;
    const double mx = wave_max(have ? rec[4] : -INFINITY);
    const double total = wave_sum(have ? rec[5] : 0.0);
    const double logN = log((double)a.N);
    const double l = wave_lse(v);
    if (lane == 0) shl[w] = l;
    __syncthreads();
    if (threadIdx.x != 0) return;
    double L[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) L[i] = shl[i];
    const int T = a.T;
    for (int i = 0; i < 3; ++i) z.log_g[(size_t)i * T + (t - 1)] = L[i];
    z.accept[t - 1] = total;
    const double rel_ess = exp(2.0 * L[1] - L[3] - logN);
    const double rel_cess = exp(-(L[2] - 2.0 * L[1] + L[0]));
    z.ess[t - 1] = rel_ess;
    // trigger 2 (SIR) resamples after every step; times fixed in advance
    // (trigger 3) run as segments and never reach this per-step merge
    const bool fire = (trigger == 0)   ? (rel_ess < nu)
                      : (trigger == 1) ? (rel_cess < nu)
                                       : (trigger == 2 && L[1] > -INFINITY);
    z.resampled[t - 1] = 0;
    z.scal[2] = 0.0;
    if (t == T) {
        z.scal[0] += L[1] - logN;
    } else if (fire) {
        z.scal[0] += L[1] - logN;
        z.scal[1] = mx;
        z.scal[2] = 1.0;
        const uint4 wd = draw_block(a.key, 0xFFFFFFFFu, (uint32_t)t, kStreamResample, 0u, 0u);
        z.scal[3] = (double)wd.x;
        z.resampled[t - 1] = 1;
        z.nres[0] += 1;
    }
}

__global__ void __launch_bounds__(kMergeThreads) k_asmc_merge(SweepArgs a, AsmcState z, int t,
                                                                int trigger, double nu)
{
    constexpr int W = kMergeThreads / kWave;
    __shared__ double shm[W][6];
    __shared__ double res[6];
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const int nb = merge_blocks(a.ntiles);
    const int64_t per = (a.ntiles + nb - 1) / nb;
    const int64_t k0 = (int64_t)blockIdx.x * per;
    const int64_t k1 = (k0 + per < a.ntiles) ? k0 + per : a.ntiles;
    // pass 1: maxima (the four log-sums and the largest log w) and the count
    double m[5] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY, -INFINITY};
    double cnt = 0.0;
    for (int64_t k = k0 + tid; k < k1; k += kMergeThreads) {
        const double* tp = z.tile_part + (size_t)k * 8;
#pragma unroll
        for (int i = 0; i < 5; ++i) m[i] = fmax(m[i], tp[i]);
        cnt += tp[5];
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) m[i] = wave_max(m[i]);
    cnt = wave_sum(cnt);
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 5; ++i) shm[w][i] = m[i];
        shm[w][5] = cnt;
    }
    __syncthreads();
    if (tid < 6) {
        double v = shm[0][tid];
        for (int ww = 1; ww < W; ++ww) v = (tid < 5) ? fmax(v, shm[ww][tid]) : v + shm[ww][tid];
        res[tid] = v;
    }
    __syncthreads();
    double M[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) M[i] = res[i];
    // pass 2: sums of exp(L_tile - max)
    double sm[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t k = k0 + tid; k < k1; k += kMergeThreads) {
        const double* tp = z.tile_part + (size_t)k * 8;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (M[i] > -INFINITY && tp[i] > -INFINITY) sm[i] += exp(tp[i] - M[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) sm[i] = wave_sum(sm[i]);
    __syncthreads();  // every thread has read res
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) shm[w][i] = sm[i];
    }
    __syncthreads();
    if (tid < 6) {
        // thread i records statistic i; its fence and the barrier stand between
        // every record and the arrival
        double* out = z.blk_part + (size_t)blockIdx.x * 8;
        if (tid < 4) {
            double acc = shm[0][tid];
            for (int ww = 1; ww < W; ++ww) acc += shm[ww][tid];
            out[tid] = lse_value(res[tid], acc);
        } else {
            out[tid] = res[tid];
        }
        __threadfence();
    }
    __syncthreads();
    // the last block to finish merges the block records; the arrival counter
    // only elects that block (no block waits for another)
    __shared__ bool last;
    if (tid == 0) last = atomicAdd(z.ticket, 1u) == (unsigned)(nb - 1);
    __syncthreads();
    if (!last) return;
    __threadfence();  // the other blocks' records
    __shared__ double shl[4];
    asmc_merge_final(a, z, t, trigger, nu, shl);
    if (tid == 0) z.ticket[0] = 0u;
}

// Merge of one segment between resampling times fixed in advance (one workgroup
// per entry, the slot order of k_merge_slots): blocks 0 .. t_end - t_begin - 1
// take the entries of steps t_begin + 1 .. t_end (moments, accepted counts; no
// per-step ESS), the last block entry T, whose log-sum-exp of the segment's
// final log-weights gives the log Z_hat factor of this event and whose fourth
// field holds the largest log w (the shift of the resampler's integer
// weights).  Each output element is written by one block.
__global__ void __launch_bounds__(kEntryThreads) k_seg_merge(SweepArgs a, AsmcState z)
{
    const int T = a.T;
    const int nsteps = a.t_end - a.t_begin;
    const bool fin = (int)blockIdx.x == nsteps;
    const int e = fin ? T : a.t_begin + (int)blockIdx.x;
    double L[3], cnt;
    __shared__ EntryShared sh;
    merge_entry(sh, a.part, a.S, T, e, L, cnt);
    double mx = -INFINITY;
    if (fin) {
        for (int64_t s = threadIdx.x; s < a.S; s += kEntryThreads)
            mx = fmax(mx, a.part[((size_t)s * (T + 1) + T) * 4 + 3]);
        mx = wave_max(mx);
        if (threadIdx.x % kWave == 0) sh.red[threadIdx.x / kWave][0] = mx;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kEntryWaves; ++u) mx = fmax(mx, sh.red[u][0]);
    }
    if (threadIdx.x != 0) return;
    if (!fin) {
#pragma unroll
        for (int i = 0; i < 3; ++i) z.log_g[(size_t)i * T + e] = L[i];
        z.accept[e] = cnt;
        z.ess[e] = NAN;
        z.resampled[e] = (e == a.t_end - 1 && a.t_end < T) ? 1 : 0;
        return;
    }
    z.scal[0] += L[0] - log((double)a.N);
    const bool fire = a.t_end < T && mx > -INFINITY && mx < INFINITY;
    z.scal[2] = fire ? 1.0 : 0.0;
    if (fire) {
        z.scal[1] = mx;
        const uint4 wd = draw_block(a.key, 0xFFFFFFFFu, (uint32_t)a.t_end, kStreamResample, 0u, 0u);
        z.scal[3] = (double)wd.x;
        z.nres[0] += 1;
    }
}

// ---------------------------------------------------------------------------
// Systematic resampling with an exact integer CDF.
//
// Bound by launches and latency, not bandwidth: 2^20 particles are 8 MB of
// log-weights in and 4 MB of ancestors out, about 3 us at the copy rate.  The
// plain call is three launches (block maxima; quantise and block-local scan;
// ancestors), every block forming the few values that span the population
// (the maximum, the prefix of the block totals) for itself instead of waiting
// for a launch of one block; a population that one workgroup's LDS holds is
// one launch.  2^20 particles: 1122 -> 61 us for the synchronous call (a single
// block of 256 threads took 1023 us for the maximum; the launches alone now
// take 37 us); 1000 particles without the synchronisation: 17.2 -> 7.6 us.
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 512;
constexpr int kScanItems = 4;
constexpr int kScanBlock = kScanThreads * kScanItems;
// Block totals that every block of the ancestor and gather kernels scans for
// itself (2^21 particles); above, one launch scans them first.
constexpr int kOwnScan = 1024;
constexpr int kAncThreads = 256;

int64_t resample_blocks(int64_t N) { return (N + kScanBlock - 1) / kScanBlock; }

__device__ __forceinline__ int quant_bits(int64_t N)
{
    int lg = 0;
    while (((int64_t)1 << lg) < N) ++lg;
    return 62 - lg;
}

// q = floor(exp(lw - max) 2^B); a NaN weight counts as zero.
__device__ __forceinline__ uint64_t quantise(double v, double mx, double scale)
{
    return (v == v) ? (uint64_t)floor(exp(v - mx) * scale) : 0;
}

// Inclusive prefix of one value per thread over the workgroup, and the total
// (integers: exact in any order).  shw: one word per wave.
template <int THREADS>
__device__ __forceinline__ uint64_t block_scan(uint64_t v, uint64_t* shw, uint64_t& total)
{
    constexpr int W = THREADS / kWave;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint64_t u = (uint64_t)__shfl_up((unsigned long long)v, o, kWave);
        if (lane >= o) v += u;
    }
    __syncthreads();  // shw may still be read from an earlier scan
    if (lane == kWave - 1) shw[w] = v;
    __syncthreads();
    uint64_t before = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        if (i < w) before += shw[i];
        total += shw[i];
    }
    return v + before;
}

// Largest value over the workgroup (NaN never enters: callers compare with >).
template <int THREADS>
__device__ __forceinline__ double block_max(double v, double* shw)
{
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) shw[w] = v;
    __syncthreads();
    double m = shw[0];
#pragma unroll
    for (int i = 1; i < THREADS / kWave; ++i) m = fmax(m, shw[i]);
    return m;
}

// Inclusive scan of the block totals, in place (one block, in chunks).
__global__ void __launch_bounds__(kScanThreads) k_rs_scan_blocks(int64_t nb, const double* scal,
                                                                 uint64_t* btot)
{
    if (scal[2] == 0.0) return;
    __shared__ uint64_t shw[kScanThreads / kWave];
    uint64_t carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
        const int64_t b = b0 + threadIdx.x;
        uint64_t total;
        const uint64_t v = block_scan<kScanThreads>((b < nb) ? btot[b] : 0, shw, total);
        if (b < nb) btot[b] = v + carry;
        carry += total;
    }
}

// The flag words of an event: largest log-weight, whether it is finite, word u.
__device__ __forceinline__ void set_event(double* scal, double mx, uint32_t u)
{
    scal[1] = mx;
    scal[2] = (mx > -INFINITY && mx < INFINITY) ? 1.0 : 0.0;
    scal[3] = (double)u;
}

// The uniform word of an event: given, or drawn for step t (particle word
// 0xFFFFFFFF, stream 3).
struct EventWord {
    uint32_t u;
    RngKey key;
    uint32_t t;
    bool draw;
};

__device__ __forceinline__ uint32_t event_word(const EventWord& e)
{
    return e.draw ? draw_block(e.key, 0xFFFFFFFFu, e.t, kStreamResample, 0u, 0u).x : e.u;
}

// Maxima of the log-weights: block b takes the blocks b, b + gridDim.x, ... of
// kScanBlock particles.
__global__ void __launch_bounds__(kScanThreads) k_rs_max(int64_t N, const double* __restrict__ lw,
                                                         double* __restrict__ bmax)
{
    __shared__ double shw[kScanThreads / kWave];
    double mx = -INFINITY;
    for (int64_t b0 = (int64_t)blockIdx.x * kScanBlock; b0 < N; b0 += (int64_t)gridDim.x * kScanBlock) {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int64_t m = b0 + k * kScanThreads + threadIdx.x;
            const double v = (m < N) ? lw[m] : -INFINITY;
            if (v > mx) mx = v;
        }
    }
    mx = block_max<kScanThreads>(mx, shw);
    if (threadIdx.x == 0) bmax[blockIdx.x] = mx;
}

// q_m and the block-local inclusive prefix into C; block totals into btot.
// With bmax (nmax maxima) the event is set here, otherwise it stands in scal.
__global__ void __launch_bounds__(kScanThreads)
    k_rs_quant_scan(int64_t N, const double* __restrict__ lw, double* scal, uint64_t* __restrict__ C,
                    uint64_t* __restrict__ btot, const double* __restrict__ bmax, int nmax,
                    EventWord ev)
{
    __shared__ uint64_t shw[kScanThreads / kWave];
    double mx;
    if (bmax) {
        mx = -INFINITY;
        for (int i = threadIdx.x; i < nmax; i += kScanThreads) mx = fmax(mx, bmax[i]);
        mx = block_max<kScanThreads>(mx, reinterpret_cast<double*>(shw));
        if (blockIdx.x == 0 && threadIdx.x == 0) set_event(scal, mx, event_word(ev));
        if (!(mx > -INFINITY && mx < INFINITY)) return;
    } else {
        if (scal[2] == 0.0) return;
        mx = scal[1];
    }
    const double scale = ldexp(1.0, quant_bits(N));
    const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
    uint64_t q[kScanItems];
    uint64_t run = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t m = base + k;
        if (m < N) run += quantise(lw[m], mx, scale);
        q[k] = run;
    }
    uint64_t total;
    const uint64_t before = block_scan<kScanThreads>(run, shw, total) - run;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t m = base + k;
        if (m < N) C[m] = before + q[k];
    }
    if (threadIdx.x == 0) btot[blockIdx.x] = total;
}

// x / N and the remainder for x / N < 2^32: a binary64 estimate (three
// roundings of a quotient below 2^32, so off by at most one) and its correction.
__device__ __forceinline__ uint64_t div_small(uint64_t x, uint64_t N, double inv_n, uint64_t& rem)
{
    uint64_t q = (uint64_t)((double)x * inv_n);
    int64_t r = (int64_t)(x - q * N);
    if (r < 0) {
        --q;
        r += (int64_t)N;
    } else if (r >= (int64_t)N) {
        ++q;
        r -= (int64_t)N;
    }
    rem = (uint64_t)r;
    return q;
}

// p_n = floor(S (2(n 2^32 + u) + 1) / (N 2^33)), S <= 2^62, n < N <= 2^30: the
// product's bits from 33 up (p < S keeps their top word below N / 4) divided
// by N as a two-digit number in base 2^32.
__device__ __forceinline__ uint64_t systematic_point(uint64_t n, uint64_t N, uint32_t u, uint64_t S,
                                                     double inv_n)
{
    const uint64_t mult = 2u * ((n << 32) | (uint64_t)u) + 1u;
    const uint64_t hi = __umul64hi(S, mult), lo = S * mult;
    const uint64_t top = hi >> 33, t = (hi << 31) | (lo >> 33);
    uint64_t rem;
    const uint64_t q1 = div_small((top << 32) | (t >> 32), N, inv_n, rem);
    const uint64_t q0 = div_small((rem << 32) | (t & 0xFFFFFFFFu), N, inv_n, rem);
    return (q1 << 32) + q0;
}

// The prefix of the block totals as the searches read it: scanned into LDS by
// this block (nb <= kOwnScan), or the global array that k_rs_scan_blocks left.
struct BlockTotals {
    uint64_t own[kOwnScan];
    uint64_t shw[kAncThreads / kWave];
};

__device__ __forceinline__ const uint64_t* block_totals(BlockTotals& sh, const uint64_t* btot,
                                                        int64_t nb)
{
    if (nb > kOwnScan) return btot;
    constexpr int per = kOwnScan / kAncThreads;
    uint64_t v[per], run = 0, total;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const int64_t b = (int64_t)threadIdx.x * per + k;
        run += (b < nb) ? btot[b] : 0;
        v[k] = run;
    }
    const uint64_t before = block_scan<kAncThreads>(run, sh.shw, total) - run;
#pragma unroll
    for (int k = 0; k < per; ++k) sh.own[threadIdx.x * per + k] = before + v[k];
    __syncthreads();
    return sh.own;
}

// Ancestor of slot n: min{m : C_m > p_n}.
__device__ __forceinline__ int64_t find_ancestor(int64_t n, int64_t N, uint32_t u, double inv_n,
                                                 const uint64_t* C, const uint64_t* btot,
                                                 int64_t nb)
{
    const uint64_t pn = systematic_point((uint64_t)n, (uint64_t)N, u, btot[nb - 1], inv_n);
    // block: first b with btot[b] > pn
    int64_t lo = 0, hi = nb - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (btot[mid] > pn) hi = mid; else lo = mid + 1;
    }
    const uint64_t off = (lo > 0) ? btot[lo - 1] : 0;
    int64_t a = lo * kScanBlock;
    int64_t b = (lo + 1) * kScanBlock - 1;
    if (b > N - 1) b = N - 1;
    while (a < b) {
        const int64_t mid = (a + b) >> 1;
        if (C[mid] + off > pn) b = mid; else a = mid + 1;
    }
    return a;
}

// Rows of `len` units copied from the rows anc[] of src to consecutive rows.
template <typename U>
__device__ __forceinline__ void gather_rows(U* __restrict__ dst, const U* __restrict__ src,
                                            const int* anc, int rows, int len)
{
    for (int e = threadIdx.x; e < rows * len; e += kAncThreads) {
        const int row = e / len;
        dst[e] = src[(size_t)anc[row] * len + (e - row * len)];
    }
}

// The event's gather: a block finds the ancestors of kGatherRows slots, one a
// thread, and then copies their rows together in the widest units that every
// row starts on (16 bytes where d allows).
constexpr int kGatherRows = 64;

__global__ void __launch_bounds__(kAncThreads) k_rs_gather(int64_t N, int d, AsmcState z, int64_t nb)
{
    if (z.scal[2] == 0.0) return;
    __shared__ BlockTotals sh;
    __shared__ int anc[kGatherRows];
    const uint32_t u = (uint32_t)z.scal[3];
    const uint64_t* bt = block_totals(sh, z.btot, nb);
    const double inv_n = 1.0 / (double)N;
    for (int64_t n0 = (int64_t)blockIdx.x * kGatherRows; n0 < N; n0 += (int64_t)gridDim.x * kGatherRows) {
        const int rows = (int)(N - n0 < kGatherRows ? N - n0 : kGatherRows);
        if ((int)threadIdx.x < rows) {
            const int64_t an = find_ancestor(n0 + threadIdx.x, N, u, inv_n, z.C, bt, nb);
            anc[threadIdx.x] = (int)an;
            z.ell2[n0 + threadIdx.x] = z.ell[an];
        }
        __syncthreads();
        float* x2 = z.X2 + (size_t)n0 * d;
        if (d % 4 == 0)
            gather_rows(reinterpret_cast<float4*>(x2), reinterpret_cast<const float4*>(z.X), anc, rows,
                        d / 4);
        else
            gather_rows(x2, (const float*)z.X, anc, rows, d);
        if (z.G) {
            double* g2 = z.G2 + (size_t)n0 * d;
            if (d % 2 == 0)
                gather_rows(reinterpret_cast<double2*>(g2), reinterpret_cast<const double2*>(z.G), anc,
                            rows, d / 2);
            else
                gather_rows(g2, (const double*)z.G, anc, rows, d);
        }
        __syncthreads();  // anc is rewritten by the next pass
    }
}

__global__ void k_rs_commit(int64_t N, int d, AsmcState z)
{
    if (z.scal[2] == 0.0) return;
    const int64_t total = N * (int64_t)d;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        z.X[i] = z.X2[i];
        if (z.G) z.G[i] = z.G2[i];
        if (i < N) {
            z.ell[i] = z.ell2[i];
            z.lw[i] = 0.0;
        }
    }
}

// Ancestors of kAncSlots consecutive slots a block.  The points increase with
// the slot, so the block's ancestors lie between those of its first and last
// slot: two waves find these (64 probes a load, three dependent loads), and
// where the range is short its part of the CDF is searched in LDS instead of
// by eleven dependent loads a slot.  39.2 us with a bitwise 128-bit division and
// a search a thread, 21.3 us now (2^20 particles, log-weights of scale 3).
// Without a finite weight every ancestor is -1 (the host call also reports it).
constexpr int kAncSlots = 1024;
constexpr int kAncRange = 2048;  // CDF entries held in LDS (24 KB with the totals: six blocks a CU)

__global__ void __launch_bounds__(kAncThreads)
    k_rs_ancestors(int64_t N, const double* scal, const uint64_t* __restrict__ C,
                   const uint64_t* __restrict__ btot, int64_t nb, int32_t* __restrict__ anc)
{
    __shared__ BlockTotals sh;
    __shared__ uint64_t cdf[kAncRange];
    __shared__ int64_t ends[2];
    const int64_t n0 = (int64_t)blockIdx.x * kAncSlots;
    const int slots = (int)(N - n0 < kAncSlots ? N - n0 : kAncSlots);
    // the totals are loaded beside the flag (without an event they are unused)
    const double flag = scal[2], word = scal[3];
    const uint64_t* bt = block_totals(sh, btot, nb);
    if (flag == 0.0) {
        for (int i = threadIdx.x; i < slots; i += kAncThreads) anc[n0 + i] = -1;
        return;
    }
    const uint32_t u = (uint32_t)word;
    const double inv_n = 1.0 / (double)N;
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (w < 2) {
        const int64_t n = w == 0 ? n0 : n0 + slots - 1;
        const uint64_t pn = systematic_point((uint64_t)n, (uint64_t)N, u, bt[nb - 1], inv_n);
        int64_t lo = 0, hi = nb - 1;  // the scan block
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (bt[mid] > pn) hi = mid; else lo = mid + 1;
        }
        const uint64_t off = lo > 0 ? bt[lo - 1] : 0;
        // entries <= p_n of the block: probes at the ends of 64 runs, then the run
        constexpr int run = kScanBlock / kWave;
        static_assert(run <= kWave, "two probes find an entry of a scan block");
        const int64_t base = lo * kScanBlock;
        const int64_t e1 = base + (int64_t)(lane + 1) * run - 1;
        const int r1 = __popcll(__ballot(e1 < N && C[e1 < N ? e1 : N - 1] + off <= pn));
        const int64_t e2 = base + (int64_t)r1 * run + lane;
        const int r2 = __popcll(__ballot(lane < run && e2 < N && C[e2 < N ? e2 : N - 1] + off <= pn));
        if (lane == 0) ends[w] = base + (int64_t)r1 * run + r2;
    }
    __syncthreads();
    const int64_t a0 = ends[0], range = ends[1] - a0 + 1;
    const bool held = range <= kAncRange;
    if (held) {
        for (int i = threadIdx.x; i < range; i += kAncThreads) {
            const int64_t b = (a0 + i) / kScanBlock;
            cdf[i] = C[a0 + i] + (b > 0 ? bt[b - 1] : 0);
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < slots; i += kAncThreads) {
        if (!held) {
            anc[n0 + i] = (int32_t)find_ancestor(n0 + i, N, u, inv_n, C, bt, nb);
            continue;
        }
        const uint64_t pn = systematic_point((uint64_t)(n0 + i), (uint64_t)N, u, bt[nb - 1], inv_n);
        int a = 0, b = (int)range - 1;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if (cdf[mid] > pn) b = mid; else a = mid + 1;
        }
        anc[n0 + i] = (int32_t)(a0 + a);
    }
}

// A population of at most kSmallN particles in one workgroup: the same
// maximum, integers and ancestors with the CDF in LDS.
constexpr int kSmallThreads = 1024;
constexpr int kSmallItems = 4;
constexpr int kSmallN = kSmallThreads * kSmallItems;

template <int ITEMS>
__global__ void __launch_bounds__(kSmallThreads)
    k_rs_small(int N, const double* __restrict__ lw, EventWord ev, double* scal,
               int32_t* __restrict__ anc)
{
    __shared__ uint64_t cdf[kSmallThreads * ITEMS];
    __shared__ uint64_t shw[kSmallThreads / kWave];
    double v[ITEMS];
    double mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int m = (int)threadIdx.x * ITEMS + k;
        v[k] = (m < N) ? lw[m] : -INFINITY;
        if (v[k] > mx) mx = v[k];
    }
    const uint32_t u = event_word(ev);
    mx = block_max<kSmallThreads>(mx, reinterpret_cast<double*>(shw));
    if (threadIdx.x == 0) set_event(scal, mx, u);
    if (!(mx > -INFINITY && mx < INFINITY)) {
        for (int n = threadIdx.x; n < N; n += kSmallThreads) anc[n] = -1;
        return;
    }
    const double scale = ldexp(1.0, quant_bits(N));
    uint64_t q[ITEMS], run = 0, S;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        run += quantise(v[k], mx, scale);  // exp(-inf) = 0 beyond N
        q[k] = run;
    }
    const uint64_t before = block_scan<kSmallThreads>(run, shw, S) - run;
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) cdf[threadIdx.x * ITEMS + k] = before + q[k];
    __syncthreads();
    const double inv_n = 1.0 / (double)N;
    for (int n = threadIdx.x; n < N; n += kSmallThreads) {
        const uint64_t pn = systematic_point((uint64_t)n, (uint64_t)N, u, S, inv_n);
        int a = 0, b = N - 1;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if (cdf[mid] > pn) b = mid; else a = mid + 1;
        }
        anc[n] = a;
    }
}

__global__ void k_philox(uint32_t k0, uint32_t k1, const uint32_t* ctr, uint32_t* out,
                         int64_t count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const uint4 c = make_uint4(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]);
    const uint4 o = philox4x32_10(c, k0, k1);
    out[4 * i] = o.x;
    out[4 * i + 1] = o.y;
    out[4 * i + 2] = o.z;
    out[4 * i + 3] = o.w;
}

// ---------------------------------------------------------------------------
// Host-side dispatch.
// ---------------------------------------------------------------------------
bool valu_shape(int d, int64_t N, ValuShape* s)
{
    if (d < 1 || d > kMaxDValu) return false;
    if (d <= 24) {
        s->lpp = 1;
        s->dpl = ((d + 3) / 4) * 4;
    } else if (d <= 32) {
        s->lpp = 2; s->dpl = 16;
    } else if (d <= 64) {
        s->lpp = 4; s->dpl = 16;
    } else if (d <= 128) {
        // 16 lanes of 8 coordinates rather than 8 of 16: half the registers
        // per lane, two waves per SIMD for the mixture/HMC sweeps (measured
        // 25% faster at d = 100)
        s->lpp = 16; s->dpl = 8;
    } else {
        s->lpp = 16; s->dpl = 16;
    }
    // Few particles: a particle on 4 lanes of 8 coordinates puts more of the
    // GPU to work (fewer lanes than two waves per SIMD otherwise)
    if (d > 8 && d <= 32 && N * s->lpp < kFillLanes) {
        s->lpp = 4;
        s->dpl = 8;
        // fewer still (4 lanes per particle would leave the SIMDs at most half
        // a wave each): 8 lanes of 4 coordinates
        if (N * 4 <= kFillLanes / 4) {
            s->lpp = 8;
            s->dpl = 4;
        }
    }
    return true;
}

int64_t valu_tiles(int64_t N, const ValuShape& s)
{
    const int64_t P = kWave / s.lpp;
    return (N + P - 1) / P;
}

template <int FAM, int MOVE>
hipError_t valu_dispatch(int what, const SweepArgs& a, const ValuShape& s, int gw,
                         const AsmcState* z, int t, hipStream_t st, const ValuBatch* b,
                         const void* ext);
static hipError_t dispatch_all(int what, const SweepArgs& a, const ValuShape& s, int gw,
                               const AsmcState* z, int t, hipStream_t st,
                               const ValuBatch* b = nullptr, const void* rj = nullptr)
{
    const int fam = a.tg.family, mv = a.move;
#define OASMC_FM(F, M) \
    if (fam == F && mv == M) return valu_dispatch<F, M>(what, a, s, gw, z, t, st, b, rj);
    OASMC_FM(kGauss, kRwmh)
    OASMC_FM(kGauss, kMala)
    OASMC_FM(kGauss, kHmc)
    OASMC_FM(kGmm, kRwmh)
    OASMC_FM(kGmm, kMala)
    OASMC_FM(kGmm, kHmc)
    OASMC_FM(kGauss, kRwmh3)
    OASMC_FM(kGmm, kRwmh3)
    OASMC_FM(kUnid, kRwmh)
    OASMC_FM(kUnid, kRwmh3)
#undef OASMC_FM
    return hipErrorInvalidValue;
}

hipError_t launch_asmc_move(const SweepArgs& a, const ValuShape& s, const AsmcState& z, int t,
                            hipStream_t st)
{
    return dispatch_all(2, a, s, 0, &z, t, st);
}

// ---------------------------------------------------------------------------
// ZJA: the online CESS-adaptive schedule of Zhou, Johansen and Aston applied
// to AIS (Sec. "Connection to online conditional ESS optimisation").  One
// workgroup chooses beta_t from log w_{t-1} and ell(X_{t-1}) of every particle:
// CESS(b) / N = g_1^2 / (g_0 g_2), g_i = sum_n w_n exp(i (b - beta_{t-1}) ell_n)
// (eq. CESS); beta_t = 1 if CESS(1) >= rho N, else `iters` halvings of
// (beta_{t-1}, 1] keeping the upper part while CESS >= rho N.  This is the
// per-step communication across all particles that the loop-swapped OAIS pass
// avoids.
//
// Bound by latency: one workgroup, so that no launch or grid barrier stands
// between two evaluations of log CESS.  Three things keep them few and short
// (2^14 particles on the Unid target, a step's choice: 742 -> 30 us):
//  * CESS(b) falls with b (log CESS has the derivative 2 (E_1 - E_2) of the mean
//    of ell under w exp(i (b - b_0) ell), which grows with i), so the halvings'
//    decisions follow from one point on either side of the crossing: a secant on
//    sqrt(-log(CESS / N)), nearly linear in b - b_0, finds the crossing, the
//    halvings are walked without evaluating, and the two ends of the last
//    interval are evaluated as they would have been.  Seven evaluations instead of
//    42; where one of the two disagrees (rounding at the crossing), the halvings go
//    on from the known points by evaluation.
//  * particles without weight (log w or ell = -inf: nine in ten on Unid) add
//    nothing, and the others are kept in LDS where they fit;
//  * one barrier an evaluation: each wave's maximum and its sum against it,
//    merged by every wave.
// ---------------------------------------------------------------------------
constexpr int kZjaThreads = 1024;
constexpr int kZjaWaves = kZjaThreads / kWave;
constexpr int kZjaHeld = 8192;  // particles held in LDS (128 KB)

// Two log-sum-exps at once from a wave's maxima m and sums s of exp against them,
// merged over the workgroup's waves (every thread ends with the same bits): row
// of 16 lanes 2 i reads the waves' entries of sum i, so the exponentials and the
// logarithm of both are formed together.  part: an entry per wave; the caller
// alternates two of them, so that one barrier separates a write from the reads
// two calls earlier.
struct ZjaPart {
    double2 v[2][kZjaWaves];
};

__device__ __forceinline__ void zja_merge(const double (&m)[2], const double (&s)[2], double (&L)[2],
                                          ZjaPart& part)
{
    static_assert(kZjaWaves == 16, "a row of 16 lanes holds one entry per wave");
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (lane < 2) part.v[lane][w] = lane == 0 ? make_double2(m[0], s[0]) : make_double2(m[1], s[1]);
    __syncthreads();
    const double2 e = part.v[lane / 32][lane % 16];
    const double M = group_max<16>(e.x);
    const double v = lse_value(M, group_sum<16>((e.x > -INFINITY) ? e.y * exp(e.x - M) : 0.0));
    L[0] = __shfl(v, 0, kWave);
    L[1] = __shfl(v, 32, kWave);
}

// log sum_n exp(log w_n), and the particles with weight into `held` in order
// while they fit (count: how many there are).  Up to 16 particles a thread are
// read once and stay in registers.
__device__ __forceinline__ double zja_gather(int64_t N, const double* __restrict__ lw,
                                             const double* __restrict__ ell, double2* held,
                                             int64_t& count, ZjaPart& part, int64_t (*cnt)[2])
{
    constexpr int kRegs = 16;
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int64_t per = (N + kZjaThreads - 1) / kZjaThreads * kWave;  // particles of a wave
    const int64_t j0 = w * per, j1 = (j0 + per < N) ? j0 + per : N;
    const bool once = per <= kRegs * kWave;
    double m[2] = {-INFINITY, -INFINITY}, s[2] = {0.0, 0.0}, L[2];
    double v[kRegs], e[kRegs];
    int64_t mine = 0, heavy = 0;  // with weight, and with log w > -inf
    auto look = [&](double lv, double le) {
        m[0] = fmax(m[0], lv);
        mine += __popcll(__ballot(lv > -INFINITY && le > -INFINITY));
        heavy += __popcll(__ballot(lv > -INFINITY));
    };
    if (once) {
#pragma unroll
        for (int k = 0; k < kRegs; ++k) {
            const int64_t j = j0 + k * kWave + lane;
            v[k] = (j < j1) ? lw[j] : -INFINITY;
            e[k] = (j < j1) ? ell[j] : -INFINITY;
        }
#pragma unroll
        for (int k = 0; k < kRegs; ++k) look(v[k], e[k]);
    } else {
        for (int64_t b = j0; b < j1; b += kWave) {
            const int64_t j = b + lane;
            look((j < j1) ? lw[j] : -INFINITY, (j < j1) ? ell[j] : -INFINITY);
        }
    }
    m[0] = group_max<kWave>(m[0]);
    if (lane == 0) {
        cnt[w][0] = mine;
        cnt[w][1] = heavy;
    }
    __syncthreads();
    int64_t at = 0, all = 0;
    count = 0;
#pragma unroll
    for (int i = 0; i < kZjaWaves; ++i) {
        if (i < w) at += cnt[i][0];
        count += cnt[i][0];
        all += cnt[i][1];
    }
    const bool fits = count <= kZjaHeld;
    // where every weight is held, the sum of the weights runs over the held
    const bool held_sum = fits && all == count;
    auto put = [&](double lv, double le) {
        const bool on = lv > -INFINITY && le > -INFINITY;
        const uint64_t bal = __ballot(on);
        if (on && fits) held[at + __popcll(bal & (((uint64_t)1 << lane) - 1))] = make_double2(lv, le);
        at += __popcll(bal);
        if (!held_sum) s[0] += (lv > -INFINITY) ? exp(lv - m[0]) : 0.0;
    };
    if (once) {
#pragma unroll
        for (int k = 0; k < kRegs; ++k) put(v[k], e[k]);
    } else {
        for (int64_t b = j0; b < j1; b += kWave) {
            const int64_t j = b + lane;
            put((j < j1) ? lw[j] : -INFINITY, (j < j1) ? ell[j] : -INFINITY);
        }
    }
    if (held_sum) {
        __syncthreads();
        m[0] = -INFINITY;
        for (int j = threadIdx.x; j < (int)count; j += kZjaThreads) m[0] = fmax(m[0], held[j].x);
        m[0] = group_max<kWave>(m[0]);
        for (int j = threadIdx.x; j < (int)count; j += kZjaThreads) s[0] += exp(held[j].x - m[0]);
    }
    s[0] = group_sum<kWave>(s[0]);
    zja_merge(m, s, L, part);
    return L[0];
}

// log sum_n exp(log w_n + i a ell_n), i = 1, 2, over the particles with weight:
// the held ones, or all of them from memory.
__device__ __forceinline__ void zja_lse(int64_t n, const double2* held, int64_t N,
                                        const double* __restrict__ lw, const double* __restrict__ ell,
                                        double a, double (&L)[2], ZjaPart& part)
{
    double m[2] = {-INFINITY, -INFINITY}, s[2] = {0.0, 0.0};
    auto pass = [&](auto&& f) {
        if (n <= kZjaHeld) {
            for (int j = threadIdx.x; j < (int)n; j += kZjaThreads) {
                const double2 v = held[j];
                f(v.x + a * v.y, v.x + 2.0 * a * v.y);
            }
        } else {
            for (int64_t j = threadIdx.x; j < N; j += kZjaThreads) {
                const double v = lw[j], e = ell[j];
                f(v + a * e, v + 2.0 * a * e);
            }
        }
    };
    pass([&](double x1, double x2) {
        m[0] = fmax(m[0], x1);
        m[1] = fmax(m[1], x2);
    });
    m[0] = group_max<kWave>(m[0]);
    m[1] = group_max<kWave>(m[1]);
    pass([&](double x1, double x2) {
        s[0] += (x1 > -INFINITY) ? exp(x1 - m[0]) : 0.0;
        s[1] += (x2 > -INFINITY) ? exp(x2 - m[1]) : 0.0;
    });
    s[0] = group_sum<kWave>(s[0]);
    s[1] = group_sum<kWave>(s[1]);
    zja_merge(m, s, L, part);
}

// The halvings of (b0, 1], the upper part kept where its start lies at most r
// from b0: the last interval (lo, hi].  A crossing estimate r between a known
// point where CESS is enough and one where it is not gives their decisions too.
__device__ __forceinline__ void zja_walk(double b0, int iters, double r, double& lo, double& hi)
{
    lo = b0;
    hi = 1.0;
    for (int it = 0; it < iters; ++it) {
        const double mid = 0.5 * (lo + hi);
        const bool up = mid - b0 <= r;
        lo = up ? mid : lo;
        hi = up ? hi : mid;
    }
}

__global__ void __launch_bounds__(kZjaThreads)
    k_zja_select(int64_t N, const double* __restrict__ lw, const double* __restrict__ ell,
                 double* beta, int t, int Tmax, double log_rho, int iters, int* stop,
                 double* log_g)
{
    if (t > *stop) return;
    extern __shared__ __align__(16) char sh_zja[];
    double2* held = reinterpret_cast<double2*>(sh_zja);
    __shared__ ZjaPart part[2];
    __shared__ int64_t cnt[kZjaWaves][2];
    const double b0 = beta[t - 1];
    const double prev = (t >= 2) ? b0 - beta[t - 2] : 1.0;
    int64_t n;
    const double L0 = zja_gather(N, lw, ell, held, n, part[0], cnt);  // fixed for the step
    double L[2], lx = -1.0;  // the moments at the offset lx
    int flip = 1;
    auto log_cess = [&](double x) {
        zja_lse(n, held, N, lw, ell, x, L, part[flip]);
        flip ^= 1;
        lx = x;
        return 2.0 * L[0] - L[1] - L0;
    };
    const double full = 1.0 - b0;
    double bt = 1.0;
    if (t < Tmax) {
        // known: enough at klo, not at khi
        double klo = 0.0, khi = INFINITY;
        const double tg = sqrt(-log_rho), cell = ldexp(full, -iters);
        double xa = 0.0, ga = 0.0, r = (prev < full) ? prev : full;
        for (int ev = 0; ev < 10; ++ev) {
            const double F = log_cess(r);
            if (F >= log_rho) {
                klo = r;
                if (r == full) break;
            } else {
                khi = r;
            }
            const double g = sqrt(fmax(-F, 0.0)), last = r;
            const bool near = fabs(g - tg) < 0.5 * tg && fabs(ga - tg) < 0.5 * tg && g != ga;
            r = near ? last + (tg - g) * (last - xa) / (g - ga) : last * tg / g;
            xa = last;
            ga = g;
            if (!(r < full) && khi == INFINITY) r = full;  // beta = 1 may be enough
            else if (!(r > klo && r < khi)) r = 0.5 * (klo + fmin(khi, full));
            if (fabs(r - last) < 0.25 * cell) break;
        }
        if (klo < full) {
            double lo, hi;
            zja_walk(b0, iters, r, lo, hi);
            // the upper end first: the lower one is the step's beta
            bool wrong = false;
            if (hi - b0 < khi) {
                wrong = log_cess(hi - b0) >= log_rho;
                if (wrong) klo = hi - b0;
                else khi = hi - b0;
            }
            if (!wrong && lo - b0 > klo) {
                wrong = !(log_cess(lo - b0) >= log_rho);
                if (wrong) khi = lo - b0;
                else klo = lo - b0;
            }
            if (wrong) {  // the known points decide what they can, evaluation the rest
                if (khi > full) khi = log_cess(full) >= log_rho ? INFINITY : full;
                lo = b0;
                hi = 1.0;
                for (int it = 0; khi <= full && it < iters; ++it) {
                    const double mid = 0.5 * (lo + hi), x = mid - b0;
                    if (x <= klo || (x < khi && log_cess(x) >= log_rho)) lo = mid;
                    else hi = mid;
                }
                bt = khi > full ? 1.0 : (lo > b0) ? lo : hi;
            } else {
                bt = (lo > b0) ? lo : hi;
            }
        }
    }
    if (lx != bt - b0) (void)log_cess(bt - b0);  // the step's moments at the chosen beta_t
    if (threadIdx.x == 0) {
        beta[t] = bt;
        log_g[t - 1] = L0;
        log_g[(size_t)Tmax + (t - 1)] = L[0];
        log_g[(size_t)2 * Tmax + (t - 1)] = L[1];
        if (bt >= 1.0) *stop = t;
    }
}

__global__ void __launch_bounds__(kZjaThreads) k_zja_final(int64_t N, const double* lw,
                                                           double* logZ)
{
    __shared__ ZjaPart part;
    double m[2] = {-INFINITY, -INFINITY}, s[2] = {0.0, 0.0}, L[2];
    for (int64_t j = threadIdx.x; j < N; j += kZjaThreads) m[0] = fmax(m[0], lw[j]);
    m[0] = group_max<kWave>(m[0]);
    for (int64_t j = threadIdx.x; j < N; j += kZjaThreads)
        s[0] += (lw[j] > -INFINITY) ? exp(lw[j] - m[0]) : 0.0;
    s[0] = group_sum<kWave>(s[0]);
    zja_merge(m, s, L, part);
    if (threadIdx.x == 0) logZ[0] = L[0] - log((double)N);
}

hipError_t launch_zja_select(int64_t N, const double* lw, const double* ell, double* beta, int t,
                             int Tmax, double log_rho, int iters, int* stop, double* log_g,
                             hipStream_t st)
{
    const size_t shb = sizeof(double2) * (size_t)std::min<int64_t>(N, kZjaHeld);
    // the attribute belongs to the process: always the largest, whatever N, so that
    // calls of several threads do not take LDS from each other
    const hipError_t e = hipFuncSetAttribute((const void*)k_zja_select,
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)(sizeof(double2) * kZjaHeld));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_zja_select, dim3(1), dim3(kZjaThreads), shb, st, N, lw, ell, beta, t, Tmax,
                       log_rho, iters, stop, log_g);
    return hipGetLastError();
}

hipError_t launch_zja_final(int64_t N, const double* lw, double* logZ, hipStream_t st)
{
    hipLaunchKernelGGL(k_zja_final, dim3(1), dim3(kZjaThreads), 0, st, N, lw, logZ);
    return hipGetLastError();
}

hipError_t launch_pt(const PtArgs& A, const ValuShape& s, hipStream_t st)
{
    return dispatch_all(5, A.a, s, 0, nullptr, 0, st, nullptr, &A);
}

hipError_t launch_rejuv(const RejuvArgs& R, const ValuShape& s, hipStream_t st)
{
    return dispatch_all(4, R.a, s, 0, nullptr, 0, st, nullptr, &R);
}

hipError_t launch_target_eval(const EvalArgs& E, const ValuShape& s, hipStream_t st)
{
    return dispatch_all(6, E.a, s, 0, nullptr, 0, st, nullptr, &E);
}

// Sum over the workgroup, in a fixed order (every thread gets it): pairwise over the
// lanes and over the waves.  (The waves one after the other leave more rounding:
// rejuvenation's averages 3.6e-16 off instead of 3.1e-16.)
template <int THREADS>
__device__ __forceinline__ double block_sum(double v, double* shw)
{
    constexpr int W = THREADS / kWave;
    v = wave_sum(v);
    __syncthreads();  // shw may still be read from an earlier sum
    if (threadIdx.x % kWave == 0) shw[threadIdx.x / kWave] = v;
    __syncthreads();
    return group_sum<W>(shw[threadIdx.x % W]);
}

// Column b of the tile sums over tiles in a fixed order.  Bound by the latency of
// the column's loads (a cache line each, few columns): a workgroup of 16 waves per
// column has them in flight at once (2^20 particles at d = 10: 85 -> 22 us).
constexpr int kColThreads = 1024;
__global__ void __launch_bounds__(kColThreads) k_rejuv_reduce(const double* __restrict__ tsum,
                                                               int64_t ntiles, int d, double samples,
                                                               double* out)
{
    __shared__ double shw[kColThreads / kWave];
    const int b = blockIdx.x;
    const int w = 2 * d + 1;
    double v = 0.0;
    for (int64_t k = threadIdx.x; k < ntiles; k += kColThreads) v += tsum[(size_t)k * w + b];
    v = block_sum<kColThreads>(v, shw);
    if (threadIdx.x == 0) out[b] = v / samples;
}

hipError_t launch_rejuv_reduce(const double* tsum, int64_t ntiles, int d, double samples,
                               double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_rejuv_reduce, dim3(2 * d + 1), dim3(kColThreads), 0, st, tsum, ntiles, d,
                       samples, out);
    return hipGetLastError();
}

// What the copies of parallel tempering leave, pooled over the copies: block n < N'
// the stepping stone of temperature n over its K T' terms (res[n]) and the summed
// rejections of pair n (res[N' + n]), block N' the round trips (res[2 N']), the
// last 2 d blocks the target chain's averages (res[2 N' + 1 ..]).  Bound by latency;
// the copies' records (8 MB for 2048 copies of 64 chains at d = 10) were pooled on
// the host before (copy, page faults and exponentials: 1.4 ms of 3.67 for 512 steps,
// now 15 us).
constexpr int kPtRedThreads = 256;
__global__ void __launch_bounds__(kPtRedThreads) k_pt_reduce(PtArgs A, int waves, double log_terms,
                                                              double samples, double* res)
{
    __shared__ double shw[kPtRedThreads / kWave];
    const int b = blockIdx.x, Np = A.Np, d = A.a.tg.d;
    double v = 0.0;
    if (b < Np) {
        double M = -INFINITY;
        for (int k = threadIdx.x; k < A.K; k += kPtRedThreads) {
            const double* o = A.out + (size_t)k * A.stride;
            if (o[2 * b + 1] > 0.0 && o[2 * b] > M) M = o[2 * b];
            v += o[2 * Np + b];
        }
        v = block_sum<kPtRedThreads>(v, shw);
        M = block_max<kPtRedThreads>(M, shw);
        double s = 0.0;
        for (int k = threadIdx.x; k < A.K; k += kPtRedThreads) {
            const double mk = A.out[(size_t)k * A.stride + 2 * b];
            const double sk = A.out[(size_t)k * A.stride + 2 * b + 1];
            if (mk > -INFINITY && sk > 0.0) s += sk * exp(mk - M);
        }
        s = block_sum<kPtRedThreads>(s, shw);
        if (threadIdx.x == 0) {
            res[b] = (s > 0.0) ? M + log(s) - log_terms : -INFINITY;
            res[Np + b] = v;
        }
        return;
    }
    if (b == Np) {
        for (int k = threadIdx.x; k < A.K; k += kPtRedThreads) v += A.out[(size_t)k * A.stride + 3 * Np];
    } else {
        const int n = A.K * waves;
        for (int e = threadIdx.x; e < n; e += kPtRedThreads)
            v += A.fpart[((size_t)(e / waves) * 16 + e % waves) * 2 * d + (b - Np - 1)];
    }
    v = block_sum<kPtRedThreads>(v, shw);
    if (threadIdx.x == 0) res[Np + b] = (b == Np) ? v : v / samples;
}

hipError_t launch_pt_reduce(const PtArgs& A, const ValuShape& s, double* res, hipStream_t st)
{
    const int P = kWave / s.lpp;
    const int waves = (A.Np + P) / P;
    hipLaunchKernelGGL(k_pt_reduce, dim3(A.Np + 1 + 2 * A.a.tg.d), dim3(kPtRedThreads), 0, st, A, waves,
                       std::log((double)A.K * A.a.T), (double)A.K * A.a.T, res);
    return hipGetLastError();
}

// One workgroup up to kSmallN particles, else three launches (four above
// kOwnScan blocks).  The line lies where the two meet: 4096 particles take
// 11.9 us in one workgroup, 8192 take 21.1 us there and 18.5 us in three launches.
static hipError_t launch_resample(int64_t N, const double* lw, const EventWord& ev, int32_t* anc,
                                  uint64_t* C, uint64_t* btot, double* scal, hipStream_t st)
{
    if (N <= kSmallThreads) {
        hipLaunchKernelGGL(k_rs_small<1>, dim3(1), dim3(kSmallThreads), 0, st, (int)N, lw, ev, scal, anc);
        return hipGetLastError();
    }
    if (N <= kSmallN) {
        hipLaunchKernelGGL(k_rs_small<kSmallItems>, dim3(1), dim3(kSmallThreads), 0, st, (int)N, lw, ev,
                           scal, anc);
        return hipGetLastError();
    }
    const int64_t nb = resample_blocks(N);
    const int nmax = (int)std::min<int64_t>(nb, kOwnScan);
    double* bmax = reinterpret_cast<double*>(btot + nb);
    hipLaunchKernelGGL(k_rs_max, dim3(nmax), dim3(kScanThreads), 0, st, N, lw, bmax);
    hipLaunchKernelGGL(k_rs_quant_scan, dim3((unsigned)nb), dim3(kScanThreads), 0, st, N, lw, scal, C,
                       btot, (const double*)bmax, nmax, ev);
    if (nb > kOwnScan)
        hipLaunchKernelGGL(k_rs_scan_blocks, dim3(1), dim3(kScanThreads), 0, st, nb,
                           (const double*)scal, btot);
    hipLaunchKernelGGL(k_rs_ancestors, dim3((unsigned)((N + kAncSlots - 1) / kAncSlots)),
                       dim3(kAncThreads), 0, st, N, (const double*)scal, (const uint64_t*)C,
                       (const uint64_t*)btot, nb, anc);
    return hipGetLastError();
}

hipError_t launch_resample_event(int64_t N, const double* lw, const RngKey& key, uint32_t t,
                                 int32_t* anc, uint64_t* C, uint64_t* btot, double* scal,
                                 hipStream_t st)
{
    return launch_resample(N, lw, EventWord{0u, key, t, true}, anc, C, btot, scal, st);
}

hipError_t launch_resample_plain(int64_t N, const double* lw, uint32_t u, int32_t* anc,
                                 uint64_t* C, uint64_t* btot, double* scal, hipStream_t st)
{
    return launch_resample(N, lw, EventWord{u, RngKey{}, 0u, false}, anc, C, btot, scal, st);
}

hipError_t launch_oais_valu_batch(int family, int move, const ValuShape& s, const ValuBatch& b,
                                  int grid_waves, hipStream_t st)
{
    SweepArgs a{};
    a.tg.family = family;
    a.move = move;
    return dispatch_all(3, a, s, grid_waves, nullptr, 0, st, &b);
}

__global__ void k_batch_params(const TargetDev* __restrict__ tgs, const BatchParam* __restrict__ bps)
{
    const TargetDev& tg = tgs[blockIdx.x];
    const BatchParam& bp = bps[blockIdx.x];
    // problems without a parameter view (logistic regression) are skipped
    if (tg.family == kLogreg || bp.m == nullptr) return;
    for (int i = threadIdx.x; i < tg.d; i += blockDim.x)
        bp.m[i] = tg.ref_mean ? tg.ref_mean[i] : 0.f;
    // 1/(2 v_k), 1/v_k; zero beyond K (padded components of a block)
    for (int k = threadIdx.x; k < kMaxK; k += blockDim.x) {
        const bool on = tg.family == kGmm && k < tg.K;
        const double v = on ? exp(2.0 * (double)tg.log_scales[k]) : 1.0;
        bp.hiv[k] = on ? 0.5 / v : 0.0;
        bp.iv[k] = on ? 1.0 / v : 0.0;
    }
    const int nl = (int)lane_param_doubles(tg, bp.lpp, bp.dpl);
    for (int e = threadIdx.x; e < nl; e += blockDim.x) bp.lane[e] = lane_param(tg, bp.lpp, bp.dpl, e);
}

hipError_t launch_batch_params(const TargetDev* tgs, const BatchParam* bp, int nprob,
                               hipStream_t st)
{
    hipLaunchKernelGGL(k_batch_params, dim3(nprob), dim3(64), 0, st, tgs, bp);
    return hipGetLastError();
}

hipError_t launch_oais_valu(const SweepArgs& a, const ValuShape& s, int grid_waves, hipStream_t st)
{
    return dispatch_all(0, a, s, grid_waves, nullptr, 0, st);
}

hipError_t launch_asmc_init(const SweepArgs& a, const ValuShape& s, const AsmcState& z,
                            hipStream_t st)
{
    return dispatch_all(1, a, s, 0, &z, 0, st);
}

hipError_t launch_asmc_step(const SweepArgs& a, const ValuShape& s, const AsmcState& z, int t,
                            int trigger, double nu, hipStream_t st)
{
    hipError_t e = dispatch_all(2, a, s, 0, &z, t, st);
    if (e != hipSuccess) return e;
    const int64_t nb = std::min<int64_t>((a.ntiles + kMergeThreads - 1) / kMergeThreads,
                                         kAsmcMergeBlocks);
    hipLaunchKernelGGL(k_asmc_merge, dim3((unsigned)nb), dim3(kMergeThreads), 0, st, a, z, t,
                       trigger, nu);
    return hipGetLastError();
}

// Grid cap of the gather and commit kernels of the resampling variant.
constexpr int64_t kIdleGrid = 2048;

hipError_t launch_resample_step(const SweepArgs& a, const AsmcState& z, int t, bool commit,
                                hipStream_t st)
{
    (void)t;
    const int64_t N = a.N;
    const int64_t nb = resample_blocks(N);
    // launched every step and idle unless the trigger fired: grids are capped
    // (grid-stride loops) so that an idle launch stays cheap
    hipLaunchKernelGGL(k_rs_quant_scan, dim3((unsigned)nb), dim3(kScanThreads), 0, st, N,
                       (const double*)z.lw, z.scal, z.C, z.btot, (const double*)nullptr, 0,
                       EventWord{});
    if (nb > kOwnScan)
        hipLaunchKernelGGL(k_rs_scan_blocks, dim3(1), dim3(kScanThreads), 0, st, nb,
                           (const double*)z.scal, z.btot);
    const int d = a.tg.d;
    const int64_t gblocks = std::min<int64_t>((N + kGatherRows - 1) / kGatherRows, kIdleGrid);
    hipLaunchKernelGGL(k_rs_gather, dim3((unsigned)gblocks), dim3(kAncThreads), 0, st, N, d, z, nb);
    if (commit) {
        const int64_t total = N * (int64_t)d;
        const int64_t blocks = std::min<int64_t>((total + 255) / 256, kIdleGrid);
        hipLaunchKernelGGL(k_rs_commit, dim3((unsigned)blocks), dim3(256), 0, st, N, d, z);
    }
    return hipGetLastError();
}

hipError_t launch_segment_merge(const SweepArgs& a, const AsmcState& z, hipStream_t st)
{
    const int nsteps = a.t_end - a.t_begin;
    hipLaunchKernelGGL(k_seg_merge, dim3(nsteps + 1), dim3(kEntryThreads), 0, st, a, z);
    return hipGetLastError();
}

hipError_t launch_merge_slots(const double* part, int64_t S, int T, int64_t N, double* log_g,
                              double* acc, double* logZ, hipStream_t st)
{
    hipLaunchKernelGGL(k_merge_slots, dim3(T + 1), dim3(kEntryThreads), 0, st, part, S, T, N, log_g, acc,
                       logZ);
    return hipGetLastError();
}

__global__ void k_zero(double* a, int na, int* b, int nb)
{
    const int i = threadIdx.x;
    if (i < na) a[i] = 0.0;
    if (i < nb) b[i] = 0;
}

hipError_t launch_zero(double* a, int na, int* b, int nb, hipStream_t st)
{
    hipLaunchKernelGGL(k_zero, dim3(1), dim3(64), 0, st, a, na, b, nb);
    return hipGetLastError();
}

hipError_t launch_philox(uint64_t seed, const uint32_t* ctr, uint32_t* out, int64_t count,
                         hipStream_t st)
{
    hipLaunchKernelGGL(k_philox, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                       (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), ctr, out, count);
    return hipGetLastError();
}

}  // namespace oasmc
