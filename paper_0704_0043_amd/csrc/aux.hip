// Auxiliary kernels: initial equilibrium, conversion between the FP64 state
// f(x, t) and the stored pre-free-flight buffer, moments, stats finalisation,
// and the storage-type dispatch of the step kernels.
#include "lbm_device.h"

namespace lbm {

hipError_t launch_step2d_st0(int, int, int, const StepArgs&, int, hipStream_t);
hipError_t launch_step2d_st1(int, int, int, const StepArgs&, int, hipStream_t);
hipError_t launch_step2d_st2(int, int, int, const StepArgs&, int, hipStream_t);
hipError_t launch_step2d_st3(int, int, int, const StepArgs&, int, hipStream_t);
hipError_t launch_step1d_st0(int, int, int, const StepArgs&, int, hipStream_t);
hipError_t launch_step1d_st1(int, int, int, const StepArgs&, int, hipStream_t);
hipError_t launch_step1d_st2(int, int, int, const StepArgs&, int, hipStream_t);
hipError_t launch_step1d_st3(int, int, int, const StepArgs&, int, hipStream_t);

hipError_t launch_step2d(int storage, int qe, int ds, int bc, const StepArgs& a, int kernel, hipStream_t s)
{
    switch (storage) {
    case kF64: return launch_step2d_st0(qe, ds, bc, a, kernel, s);
    case kF32: return launch_step2d_st1(qe, ds, bc, a, kernel, s);
    case kF16: return launch_step2d_st2(qe, ds, bc, a, kernel, s);
    case kBF16: return launch_step2d_st3(qe, ds, bc, a, kernel, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_step1d(int storage, int qe, int ds, int bc, const StepArgs& a, int kernel, hipStream_t s)
{
    switch (storage) {
    case kF64: return launch_step1d_st0(qe, ds, bc, a, kernel, s);
    case kF32: return launch_step1d_st1(qe, ds, bc, a, kernel, s);
    case kF16: return launch_step1d_st2(qe, ds, bc, a, kernel, s);
    case kBF16: return launch_step1d_st3(qe, ds, bc, a, kernel, s);
    }
    return hipErrorInvalidValue;
}

// one workgroup per domain: the sums of the step just run
__global__ void __launch_bounds__(kThreads) k_finalize(StepArgs a, long long step)
{
    __shared__ double red[kThreads];
    reduce_domain(a, a.dom[blockIdx.x], a.median_pass, step, red);
}

// D2Q9: the set-0 partial of each group is the sum of the collision partials
// of its workgroups, in order.
__global__ void __launch_bounds__(kThreads) k_group_sums(StepArgs a)
{
    __shared__ double buf[kGroupParts * kNStat + 8 * kNStat];
    const Group t = a.groups[blockIdx.x];
    const long long p0 = (long long)a.dom[t.domain].part_first + t.n0 / kThreads;
    sum_partials(a.partials + (long long)blockIdx.x * kNStat, a.blockpart + p0 * kNStat,
                 (t.n1 - t.n0 + kThreads - 1) / kThreads, buf);
}

// E(Delta S') of this step and the thresholds of the ensemble limiters, per
// domain (Sec. 3.3, 3.4): the collision partials (set 0; for D2Q9 summed per
// group beforehand) are reduced exactly as the stats are, so E equals the
// reported mean_dS bit for bit.
__global__ void __launch_bounds__(kThreads) k_ens_prepare(StepArgs a)
{
    __shared__ double red[kThreads];
    const DomainDev& D = a.dom[blockIdx.x];
    if (!(D.limiter & kLimEns)) return;
    reduce_domain(a, D, false, a.counter[a.parity], red);
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double nf = D.stats[kSFluid];
    const double mean = nf > 0.0 ? D.stats[kSDpost] / nf : 0.0;
    D.ens[kEMean] = mean;
    D.ens[kEThresh] = fmax(D.ens_c * mean, D.delta_ens);
    D.ens[kESmoothA] = mean > 0.0 ? D.delta_ens / pow(mean, D.ens_k) : 0.0;
    if (D.limiter & kLimEnsBudget) {
        // eq. (EntThresh): the limiter may produce delta_0 times the
        // entropy production of the LBGK step, [1 - (2 beta - 1)^2] sum Delta S
        BudgetState& b = *D.bstate;
        const double budget = D.ens_c * (1.0 - D.c * D.c) * D.stats[kSDpost];
        b.prefix = 0;
        b.budget = budget;
        b.s_above = 0.0;
        b.c_above = 0.0;
        b.level = 0;
        b.done = budget > 0.0 ? 0 : 1;
        // no budget: the threshold sits at the largest value, nothing moves
        D.ens[kEBudget] = fmax(budget > 0.0 ? 0.0 : D.stats[kSMax], D.delta_ens);
    }
    if (D.limiter & kLimTopK) {
        // top-k trimming (Sec. 3.2): the k-th largest finite Delta S' by the
        // same radix selection, counts only; -inf (every node above
        // delta) until found
        BudgetState& b = *D.bstate;
        b.prefix = 0;
        b.budget = double(D.top_k);
        b.s_above = 0.0;
        b.c_above = 0.0;
        b.level = 0;
        b.done = 0;
        D.ens[kETopk] = -__builtin_huge_val();
    }
}

// Keys of the budget selection: the bit pattern of a non-negative finite
// value (0 for values <= 0), ordered as the values are.
template <class A>
struct BKey;
template <>
struct BKey<double> {
    using U = unsigned long long;
    static constexpr bool dbl = true;
    static constexpr int mbits = 52, bias = 1075;
    __device__ static U key(double d) { return d > 0.0 ? U(__double_as_longlong(d)) : U(0); }
    __device__ static double value(U k) { return __longlong_as_double((long long)k); }
};
template <>
struct BKey<float> {
    using U = unsigned int;
    static constexpr bool dbl = false;
    static constexpr int mbits = 23, bias = 150;
    __device__ static U key(float d) { return d > 0.0f ? U(__float_as_uint(d)) : U(0); }
    __device__ static double value(U k) { return double(__uint_as_float(k)); }
};

// integer significand m and exponent e of a key: value = m 2^e
template <class K>
__device__ inline unsigned long long key_significand(typename K::U k)
{
    using U = typename K::U;
    const U e = k >> K::mbits;
    return (unsigned long long)((k & ((U(1) << K::mbits) - 1)) | (e ? (U(1) << K::mbits) : U(0)));
}
template <class K>
__device__ inline int key_exponent(typename K::U k)
{
    const int e = int(k >> K::mbits);
    return (e ? e : 1) - K::bias;
}

// One level of the budget selection: a histogram of the digit (count and exact
// significand sum per bucket) of the values whose higher digits match the
// prefix, added into the domain's histogram.  A workgroup of 1024 threads
// takes a run of groups (16384 consecutive nodes each): what a level costs are the additions
// of all workgroups to the few buckets that most values share, which queue at
// their addresses (1000 workgroups: 40 us for the first level of a 1024 x 1000
// grid, against 12 us with 64), so workgroups are few and large.  Each thread
// takes 16 nodes of a group, one of every 1024, and merges runs of equal buckets
// in registers first (the significand sum of a wave stays below 2^63).
constexpr int kHistThreads = 1024, kHistBlocks = 256;
template <class A, bool CAV>
__global__ void __launch_bounds__(kHistThreads) k_budget_hist(StepArgs a, int level)
{
    using K = BKey<A>;
    using U = typename K::U;
    __shared__ unsigned hn[kBudgetBuckets];
    __shared__ unsigned long long hlo[kBudgetBuckets];
    __shared__ unsigned hhi[kBudgetBuckets];
    const int tid = int(threadIdx.x), lane = tid & (kWave - 1);
    const int lo = budget_lo(K::dbl, level), hi = budget_hi(K::dbl, level);
    const U dmask = (U(1) << (hi - lo)) - 1;
    for (int k = tid; k < kBudgetBuckets; k += kHistThreads) {
        hn[k] = 0;
        hlo[k] = 0;
        hhi[k] = 0;
    }
    __syncthreads();
    auto flush = [&](int b, unsigned cnt, unsigned long long sum) {
        atomicAdd(&hn[b], cnt);
        const unsigned long long old = atomicAdd(&hlo[b], sum);
        if (old + sum < old) atomicAdd(&hhi[b], 1u);
    };
    // Neighbouring columns mostly hold values of one binary exponent: in the
    // first level their 64 additions to one bucket would queue at one LDS
    // address, so the lanes that share the first flushing lane's bucket are
    // added up first.  Lanes take part with cnt = 0 when they have nothing.
    auto flush_wave = [&](int b, unsigned cnt, unsigned long long sum) {
        const unsigned long long have = __ballot(cnt != 0);
        if (!have) return;
        const int lead = __shfl(b, __builtin_ctzll(have), kWave);
        const bool same = cnt != 0 && b == lead;
        unsigned c = same ? cnt : 0u;
        unsigned long long v = same ? sum : 0ull;
#pragma unroll
        for (int off = kWave / 2; off >= 1; off >>= 1) {
            c += __shfl_xor(c, off, kWave);
            v += __shfl_xor(v, off, kWave);
        }
        if (lane == 0) flush(lead, c, v);
        if (cnt && !same) flush(b, cnt, sum);
    };
    const int nb = int(gridDim.x), g0 = int((long long)blockIdx.x * a.ngroups / nb),
              g1 = int((long long)(blockIdx.x + 1) * a.ngroups / nb);
    for (int g = g0; g < g1; ++g) {
        const Group t = a.groups[g];
        const DomainDev& D = a.dom[t.domain];
        bool run = D.limiter & (kLimEnsBudget | kLimTopK);
        if (run) {
            // the first nodes are on their way before `done` is looked at
            const int done = D.bstate->done;
            const unsigned long long prefix = D.bstate->prefix;
            run = !done;
            const A* ds = static_cast<const A*>(D.dsbuf);
            int cur = -1;
            unsigned cnt = 0;
            unsigned long long sum = 0;
            constexpr int kAhead = 8;      // nodes loaded together
            for (int n = t.n0 + tid; n < t.n1; n += kAhead * kHistThreads) {
                A v[kAhead];
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
                    const int nk = n + k * kHistThreads;
                    v[k] = nk < t.n1 ? ds[nk] : A(__builtin_huge_val());
                }
                if (done) break;
#pragma unroll
                for (int k = 0; k < kAhead; ++k) {
                    if (!isfinite(v[k])) continue;
                    if (CAV) {
                        const int nk = n + k * kHistThreads, y = nk / D.nx, x = nk - y * D.nx;
                        if (x == 0 || x == D.nx - 1 || y == 0 || y == D.ny - 1) continue;   // walls and lid
                    }
                    const U key = K::key(v[k]);
                    if ((unsigned long long)(key >> hi) != prefix) continue;
                    const int b = int((key >> lo) & dmask);
                    if (b != cur) {
                        if (cnt) flush(cur, cnt, sum);
                        cur = b;
                        cnt = 0;
                        sum = 0;
                    }
                    ++cnt;
                    sum += key_significand<K>(key);
                }
            }
            if (!run) continue;
            if (level == 0) flush_wave(cur, cnt, sum);
            else if (cnt) flush(cur, cnt, sum);
        }
        // into the domain's histogram after its last group here
        if (run && (g + 1 == g1 || a.groups[g + 1].domain != t.domain)) {
            __syncthreads();
            BudgetBucket* gh = D.bhist;
            for (int k = tid; k < kBudgetBuckets; k += kHistThreads)
                if (hn[k]) {
                    atomicAdd(&gh[k].n, (unsigned long long)hn[k]);
                    const unsigned long long old = atomicAdd(&gh[k].lo, hlo[k]);
                    const unsigned long long hiadd = (unsigned long long)hhi[k] + (old + hlo[k] < old ? 1ull : 0ull);
                    if (hiadd) atomicAdd(&gh[k].hi, hiadd);
                    hn[k] = 0;
                    hlo[k] = 0;
                    hhi[k] = 0;
                }
            __syncthreads();
        }
    }
}

// Exclusive sums over the threads above (tid + 1 .. kThreads - 1) of one or two
// values per thread, plus a start value: a shuffle scan in each wave, then the
// totals of the waves above.  (One thread adding 256 LDS values in turn took
// 10 of the 15 us of a select launch.)
template <int N>
__device__ inline void sums_above(double (&v)[N], const double (&start)[N], double* lds /* [kThreads / kWave * N] */)
{
    const int lane = int(threadIdx.x) & (kWave - 1), wave = int(threadIdx.x) / kWave;
    constexpr int nw = kThreads / kWave;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1)
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const double o = __shfl_down(v[k], off, kWave);
            if (lane + off < kWave) v[k] += o;
        }
    // (the next lane's sum: taking the own value off this lane's would lose the
    // digits of few large values above many small ones)
    double above[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double o = __shfl_down(v[k], 1, kWave);
        above[k] = lane + 1 < kWave ? o : 0.0;
    }
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) lds[wave * N + k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        double s = start[k];
        for (int w = nw - 1; w > wave; --w) s += lds[w * N + k];
        v[k] = s + above[k];
    }
}

// One level of the budget selection, one workgroup per domain.  With
// g(t) = sum over values v > t of (v - t), decreasing in t, the threshold
// solves g(Delta S_0) = budget; it lies in the highest bucket whose lower
// edge L has g(L) >= budget.  That bucket's digit extends the prefix; at the
// last level the bucket is a single value v, g is linear above it, and
// Delta S_0 = (sum of the values above v - budget) / (their count).  The
// histogram is read in a fixed order and left zero for the next level.
template <class A>
__global__ void __launch_bounds__(kThreads) k_budget_select(StepArgs a, int level)
{
    using K = BKey<A>;
    using U = typename K::U;
    constexpr int per = kBudgetBuckets / kThreads;
    __shared__ double waves[2 * kThreads / kWave];
    __shared__ int best;
    const DomainDev& D = a.dom[blockIdx.x];
    if (!(D.limiter & kLimEnsBudget)) return;
    BudgetState* bs = D.bstate;
    const int tid = int(threadIdx.x);
    // the state and the buckets come together, not one after the other
    const int done = bs->done;
    const unsigned long long prefix = bs->prefix;
    const double budget = bs->budget;
    const double start[2] = {bs->s_above, bs->c_above};
    BudgetBucket g[per];
#pragma unroll
    for (int i = 0; i < per; ++i) g[i] = D.bhist[tid * per + i];
    if (done) return;
    const int lo = budget_lo(K::dbl, level), hi = budget_hi(K::dbl, level);
    const int w = hi - lo;
    auto edge_of = [&](int b) { return U(((prefix << w) | (unsigned long long)b) << lo); };
    double s[per], c[per];
    double my_s = 0.0, my_c = 0.0;
#pragma unroll
    for (int i = per - 1; i >= 0; --i) {
        const int b = tid * per + i;
        BudgetBucket& gb = D.bhist[b];
        const unsigned long long n = g[i].n, l = g[i].lo, h = g[i].hi;
        gb.n = 0;
        gb.lo = 0;
        gb.hi = 0;
        c[i] = double(n);
        s[i] = n ? ldexp(double(h) * 18446744073709551616.0 + double(l), key_exponent<K>(edge_of(b))) : 0.0;
        my_s += s[i];
        my_c += c[i];
    }
    if (tid == 0) best = -1;
    double above[2] = {my_s, my_c};
    sums_above<2>(above, start, waves);
    const int nb = 1 << w;   // buckets of this digit (the rest stay empty)
    double S = above[0], C = above[1];
    double sa = 0.0, ca = 0.0, sa0 = 0.0, ca0 = 0.0;
    int mine = -1;
#pragma unroll
    for (int i = per - 1; i >= 0; --i) {
        const int b = tid * per + i;
        const double L = b < nb ? K::value(edge_of(b)) : 0.0;
        if (i == 0) {
            sa0 = S;
            ca0 = C;
        }
        const double S1 = S + s[i], C1 = C + c[i];
        if (mine < 0 && b < nb && S1 - L * C1 >= budget) {
            mine = b;
            sa = S;
            ca = C;
        }
        S = S1;
        C = C1;
    }
    if (mine >= 0) atomicMax(&best, mine);
    __syncthreads();
    int j = best;
    if (j < 0 && level == 0) {
        // the budget exceeds g(0) = sum Delta S: every node goes to f*
        if (tid == 0) {
            D.ens[kEBudget] = fmax(0.0, D.delta_ens);
            bs->done = 1;
        }
        return;
    }
    if (j < 0) {
        // the lower edge of the parent bucket met the condition; rounding in
        // the regrouped sums may put it just below here: keep its lowest bucket
        j = 0;
        mine = tid == 0 ? 0 : -1;
        sa = sa0;
        ca = ca0;
    }
    if (mine != j) return;
    bs->prefix = (prefix << w) | (unsigned long long)j;
    bs->s_above = sa;
    bs->c_above = ca;
    bs->level = level + 1;
    if (level + 1 == budget_levels(K::dbl)) {
        const double v = K::value(edge_of(j));
        const double t0 = ca > 0.0 ? (sa - budget) / ca : v;
        D.ens[kEBudget] = fmax(fmax(t0, 0.0), D.delta_ens);
        bs->done = 1;
    }
}

// One level of the top-k selection, one workgroup per domain: the bucket
// holding the k-th largest value is the highest one where the count of the
// values at or above its lower edge reaches k.  At the last level the bucket
// is a single value, the k-th largest; trimming acts at and above it (ties
// included).  Fewer than k finite values: every node above delta.
template <class A>
__global__ void __launch_bounds__(kThreads) k_topk_select(StepArgs a, int level)
{
    using K = BKey<A>;
    using U = typename K::U;
    constexpr int per = kBudgetBuckets / kThreads;
    __shared__ double waves[kThreads / kWave];
    __shared__ int best;
    const DomainDev& D = a.dom[blockIdx.x];
    if (!(D.limiter & kLimTopK)) return;
    BudgetState* bs = D.bstate;
    const int tid = int(threadIdx.x);
    const int done = bs->done;
    const unsigned long long prefix = bs->prefix;
    const double kk = bs->budget;
    const double start[1] = {bs->c_above};
    unsigned long long n[per];
#pragma unroll
    for (int i = 0; i < per; ++i) n[i] = D.bhist[tid * per + i].n;
    if (done) return;
    const int lo = budget_lo(K::dbl, level), hi = budget_hi(K::dbl, level);
    const int w = hi - lo;
    const int nb = 1 << w;
    double c[per];
    double my_c = 0.0;
#pragma unroll
    for (int i = per - 1; i >= 0; --i) {
        BudgetBucket& gb = D.bhist[tid * per + i];
        c[i] = double(n[i]);
        gb.n = 0;
        gb.lo = 0;
        gb.hi = 0;
        my_c += c[i];
    }
    if (tid == 0) best = -1;
    double above[1] = {my_c};
    sums_above<1>(above, start, waves);
    double C = above[0], ca = 0.0, ca0 = 0.0;
    int mine = -1;
#pragma unroll
    for (int i = per - 1; i >= 0; --i) {
        const int b = tid * per + i;
        if (i == 0) ca0 = C;
        const double C1 = C + c[i];
        if (mine < 0 && b < nb && C1 >= kk) {
            mine = b;
            ca = C;
        }
        C = C1;
    }
    if (mine >= 0) atomicMax(&best, mine);
    __syncthreads();
    int j = best;
    if (j < 0 && level == 0) {
        if (tid == 0) bs->done = 1;      // fewer than k values: no limit
        return;
    }
    if (j < 0) {
        j = 0;
        mine = tid == 0 ? 0 : -1;
        ca = ca0;
    }
    if (mine != j) return;
    const U edge = U(((prefix << w) | (unsigned long long)j) << lo);
    bs->prefix = (prefix << w) | (unsigned long long)j;
    bs->c_above = ca;
    bs->level = level + 1;
    if (level + 1 == budget_levels(K::dbl)) {
        D.ens[kETopk] = K::value(edge);
        bs->done = 1;
    }
}

template <class A>
static hipError_t budget_levels_t(int bc, const StepArgs& a, hipStream_t s)
{
    for (int level = 0; level < budget_levels(sizeof(A) == 8); ++level) {
        const dim3 grid(a.ngroups < kHistBlocks ? a.ngroups : kHistBlocks), block(kHistThreads);
        if (bc == kCavity)
            hipLaunchKernelGGL((k_budget_hist<A, true>), grid, block, 0, s, a, level);
        else
            hipLaunchKernelGGL((k_budget_hist<A, false>), grid, block, 0, s, a, level);
        if (a.budget & kSelectBudget)
            hipLaunchKernelGGL(k_budget_select<A>, dim3(a.ndomains), dim3(kThreads), 0, s, a, level);
        if (a.budget & kSelectTopK)
            hipLaunchKernelGGL(k_topk_select<A>, dim3(a.ndomains), dim3(kThreads), 0, s, a, level);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_budget(int storage, int bc, const StepArgs& a, hipStream_t s)
{
    return storage == kF64 ? budget_levels_t<double>(bc, a, s) : budget_levels_t<float>(bc, a, s);
}

hipError_t launch_ens_prepare(const StepArgs& a, hipStream_t s)
{
    if (a.nblocks > 0) {
        hipLaunchKernelGGL(k_group_sums, dim3(a.ngroups), dim3(kThreads), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_ens_prepare, dim3(a.ndomains), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_finalize(const StepArgs& a, long long steps_done, hipStream_t s)
{
    if (a.nblocks > 0 && !a.fused) {
        hipLaunchKernelGGL(k_group_sums, dim3(a.ngroups), dim3(kThreads), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_finalize, dim3(a.ndomains), dim3(kThreads), 0, s, a, steps_done);
    return hipGetLastError();
}

// The number of nodes the median filter moved in the step just run:
// the sum of the second-pass partials (set 1) of every tile,
// which the two kernels and the fused step both write.  One workgroup, a
// fixed order of the sums.
__global__ void __launch_bounds__(kThreads) k_filtered_count(StepArgs a, double* out)
{
    __shared__ double red[kThreads];
    const double* part = a.partials + (long long)a.pstride * kNStat;
    double s = 0.0;
    for (int t = int(threadIdx.x); t < a.ntiles; t += kThreads) s += part[(long long)t * kNStat + kSFilt];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w /= 2) {
        if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

hipError_t launch_filtered_count(const StepArgs& a, double* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_filtered_count, dim3(1), dim3(kThreads), 0, s, a, out);
    return hipGetLastError();
}

// f = f*(rho, u) at every node, FP64 (Sec. 4.1 quasiequilibria)
template <int LAT, int QE>
__global__ void k_init_f(const double* __restrict__ rho, const double* __restrict__ u, double* __restrict__ f,
                         int n)
{
    using L = Lat<LAT>;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const double r = rho[s];
    const double ux = u[s];
    const double uy = LAT == kD2Q9 ? u[n + s] : 0.0;
    double E[L::Q];
    eq_excess<LAT, QE>(ux, uy, E);
#pragma unroll
    for (int i = 0; i < L::Q; ++i) f[(long long)i * n + s] = r * L::w(i) * (1.0 + E[i]);
}

hipError_t launch_init_f(int lattice, int qe, const double* rho, const double* u, double* f, int nx, int ny,
                         hipStream_t s)
{
    const int n = nx * ny;
    const dim3 grid((n + 255) / 256), block(256);
    if (lattice == kD2Q9) {
        if (qe == kPoly) hipLaunchKernelGGL((k_init_f<kD2Q9, kPoly>), grid, block, 0, s, rho, u, f, n);
        else hipLaunchKernelGGL((k_init_f<kD2Q9, kEntropic>), grid, block, 0, s, rho, u, f, n);
    } else {
        if (qe == kPoly) hipLaunchKernelGGL((k_init_f<kD1Q3, kPoly>), grid, block, 0, s, rho, u, f, n);
        else hipLaunchKernelGGL((k_init_f<kD1Q3, kEntropic>), grid, block, 0, s, rho, u, f, n);
    }
    return hipGetLastError();
}

// The buffer holds the values o_i(x) about to leave x; the state is
// f_i(x) = o_i(x - v_i) (or o_opp(i)(x) off a non-periodic edge).  Scatter
// inverts that map: o_i(x) = f_i(x + v_i), or f_opp(i)(x) when x + v_i is off
// the grid.
template <int LAT, class T>
__global__ void k_scatter(const double* __restrict__ f, T* buf_, long long plane, int nx, int ny,
                          int periodic, double shift)
{
    using L = Lat<LAT>;
    const gptr<T> buf = to_global<T>(static_cast<void*>(buf_));
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    const int n = nx * ny;
    if (s >= n) return;
    const int x = s % nx, y = s / nx;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        int tx = x + L::vx(i), ty = y + L::vy(i);
        double v;
        if (periodic) {
            tx = wrapi(tx, nx);
            ty = wrapi(ty, ny);
            v = f[(long long)i * n + ty * nx + tx];
        } else if (tx >= 0 && tx < nx && ty >= 0 && ty < ny) {
            v = f[(long long)i * n + ty * nx + tx];
        } else {
            v = f[(long long)L::opp(i) * n + s];
        }
        Store<T>::st(buf + i * plane + s, typename Store<T>::A(v - L::w(i) * shift));
    }
}

// Gather: f_i(x) from the buffer as FP64; optionally rho and u (eq. macro_dis)
template <int LAT, class T>
__global__ void k_gather(const T* buf_, long long plane, double* __restrict__ f, int nx, int ny,
                         int periodic, double shift, int want_f, double* __restrict__ rho, double* __restrict__ u)
{
    using L = Lat<LAT>;
    const gptr<const T> buf = to_global<T>(static_cast<const void*>(buf_));
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    const int n = nx * ny;
    if (s >= n) return;
    const int x = s % nx, y = s / nx;
    double r = 0, jx = 0, jy = 0;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        int sx = x - L::vx(i), sy = y - L::vy(i);
        long long off;
        if (periodic) {
            off = i * plane + wrapi(sy, ny) * nx + wrapi(sx, nx);
        } else if (sx >= 0 && sx < nx && sy >= 0 && sy < ny) {
            off = i * plane + sy * nx + sx;
        } else {
            off = L::opp(i) * plane + s;
        }
        const double v = double(Store<T>::ld(buf + off)) + L::w(i) * shift;
        if (want_f) f[(long long)i * n + s] = v;
        r += v;
        jx += L::vx(i) * v;
        jy += L::vy(i) * v;
    }
    if (rho) rho[s] = r;
    if (u) {
        u[s] = jx / r;
        if (LAT == kD2Q9) u[n + s] = jy / r;
    }
}

template <class T>
static hipError_t scatter_t(int lattice, int periodic, const double* f, void* buf, long long plane, int nx, int ny,
                            double shift, hipStream_t s)
{
    const int n = nx * ny;
    const dim3 grid((n + 255) / 256), block(256);
    if (lattice == kD2Q9)
        hipLaunchKernelGGL((k_scatter<kD2Q9, T>), grid, block, 0, s, f, (T*)buf, plane, nx, ny, periodic, shift);
    else
        hipLaunchKernelGGL((k_scatter<kD1Q3, T>), grid, block, 0, s, f, (T*)buf, plane, nx, ny, periodic, shift);
    return hipGetLastError();
}

template <class T>
static hipError_t gather_t(int lattice, int periodic, const void* buf, long long plane, double* f, int nx, int ny,
                           double shift, int want_f, double* rho, double* u, hipStream_t s)
{
    const int n = nx * ny;
    const dim3 grid((n + 255) / 256), block(256);
    if (lattice == kD2Q9)
        hipLaunchKernelGGL((k_gather<kD2Q9, T>), grid, block, 0, s, (const T*)buf, plane, f, nx, ny, periodic, shift,
                           want_f, rho, u);
    else
        hipLaunchKernelGGL((k_gather<kD1Q3, T>), grid, block, 0, s, (const T*)buf, plane, f, nx, ny, periodic, shift,
                           want_f, rho, u);
    return hipGetLastError();
}

hipError_t launch_scatter(int storage, int lattice, int bc, const double* f, void* buf, long long plane, int nx,
                          int ny, double shift, hipStream_t s)
{
    const int periodic = bc == kPeriodic;
    switch (storage) {
    case kF64: return scatter_t<double>(lattice, periodic, f, buf, plane, nx, ny, shift, s);
    case kF32: return scatter_t<float>(lattice, periodic, f, buf, plane, nx, ny, shift, s);
    case kF16: return scatter_t<_Float16>(lattice, periodic, f, buf, plane, nx, ny, shift, s);
    case kBF16: return scatter_t<__bf16>(lattice, periodic, f, buf, plane, nx, ny, shift, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gather(int storage, int lattice, int bc, const void* buf, long long plane, double* f, int nx, int ny,
                         double shift, int want_f, double* rho, double* u, hipStream_t s)
{
    const int periodic = bc == kPeriodic;
    switch (storage) {
    case kF64: return gather_t<double>(lattice, periodic, buf, plane, f, nx, ny, shift, want_f, rho, u, s);
    case kF32: return gather_t<float>(lattice, periodic, buf, plane, f, nx, ny, shift, want_f, rho, u, s);
    case kF16: return gather_t<_Float16>(lattice, periodic, buf, plane, f, nx, ny, shift, want_f, rho, u, s);
    case kBF16: return gather_t<__bf16>(lattice, periodic, buf, plane, f, nx, ny, shift, want_f, rho, u, s);
    }
    return hipErrorInvalidValue;
}

// `words` 32-bit words of a ring of `cap`, from word `first` on, to pinned host
// memory.  A few KB by this kernel and a wait take 13 us, where a copy into
// pageable memory takes 35.
__global__ void k_read(const unsigned* __restrict__ ring, unsigned* __restrict__ out, int words, int first, int cap)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= words) return;
    int at = first + k;
    if (at >= cap) at -= cap;
    out[k] = ring[at];
}

// needs 0 <= first < cap and words <= cap
hipError_t launch_read(const void* ring, void* out, int words, int first, int cap, hipStream_t s)
{
    hipLaunchKernelGGL(k_read, dim3((words + 255) / 256), dim3(256), 0, s, static_cast<const unsigned*>(ring),
                       static_cast<unsigned*>(out), words, first, cap);
    return hipGetLastError();
}

}  // namespace lbm
