// kb_rung.hip -- the rung benchmarker's statistics over timing samples.
//
// A rung times every surviving candidate on the rung's shapes, a number of
// iterations each (Section 3.2: fidelity level and rung budget; Appendix
// A.2: 4, 16 and 60 iterations on three rungs).  From those samples the
// scheduler needs, per (candidate, shape) row, the mean time and the speedup
// over the baseline (Appendix A.5), the quantiles behind the tail ratios of
// Table A.3, and per candidate the latency and the runtime score of Eq. 2.
//
// rung_kernel        rows of at most 256 samples (every rung of the paper):
//                    one work-group per candidate, one wave per row, up to 4
//                    samples per lane, a bitonic sort across lanes and
//                    registers, then the candidate's score (or rows only);
// rows_block_kernel  longer rows (up to kRungMaxIter), and rows of more than
//                    128 samples where there are few: one work-group per row,
//                    bitonic sort in LDS;
// scores_kernel      after rows alone, one thread per candidate: latency,
//                    score, speedups (which way is taken: launch_rung_stats);
// promote_kernel     the promotion decision over the scores.
//
// Every sum runs left to right in binary64, as the definitions read (the
// rows are short, so a sequential sum costs little), and every formula is
// evaluated with explicit roundings in the order written, so the results are
// the same bits as the definition's.
#include "kb_device.hpp"
#include "kb_internal.hpp"
#include "kb_rung.hpp"

namespace kb {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ bool sample_ok(double t) { return __builtin_isfinite(t) && t > 0.0; }

// The p-quantile of x sorted ascending (n >= 1): linear interpolation
// between the order statistics around position h = (n - 1) p.
template <class Get>
__device__ __forceinline__ double quantile(Get x, int n, double p) {
    const double h = __dmul_rn((double)(n - 1), p);
    const int k = (int)floor(h);
    if (k >= n - 1) return x(n - 1);
    const double t = __dsub_rn(h, (double)k);
    const double a = x(k), b = x(k + 1);
    return __dadd_rn(a, __dmul_rn(t, __dsub_rn(b, a)));
}

__device__ __forceinline__ void write_row(kb_sample_stats* o, int n, bool valid, double sum,
                                          double q50, double q90, double q95, double q99) {
    kb_sample_stats r;
    const double nan = __builtin_nan("");
    r.n_samples = n;
    r.valid = valid ? 1 : 0;
    r.speedup_vs_base = nan;  // set by scores_kernel
    if (valid) {
        r.mean_us = sum / (double)n;
        r.p50_us = q50;
        r.p90_us = q90;
        r.p95_us = q95;
        r.p99_us = q99;
        r.p90_over_p50 = q90 / q50;
        r.p95_over_p50 = q95 / q50;
        r.p99_over_p50 = q99 / q50;
    } else {
        r.mean_us = r.p50_us = r.p90_us = r.p95_us = r.p99_us = nan;
        r.p90_over_p50 = r.p95_over_p50 = r.p99_over_p50 = nan;
    }
    *o = r;
}

// The 64-bit value of lane ^ M: one DPP permutation inside a row of 16 lanes
// (two for M = 4), a bpermute across rows.
template <int M>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v) {
    if constexpr (M == 1) return dpp_u64<DPP_QUAD_XOR1>(v);
    else if constexpr (M == 2) return dpp_u64<DPP_QUAD_XOR2>(v);
    else if constexpr (M == 3) return dpp_u64<0x1B>(v);  // quad_perm [3, 2, 1, 0]
    else if constexpr (M == 7) return dpp_u64<DPP_ROW_HALF_MIRROR>(v);
    else if constexpr (M == 15) return dpp_u64<DPP_ROW_MIRROR>(v);
    else if constexpr (M == 4) return lane_xor<3>(lane_xor<7>(v));
    else if constexpr (M == 8) return dpp_u64<0x128>(v);  // row_ror:8
    else return __shfl_xor((unsigned long long)v, M, 64);
}

// v[e] at lane l is element 64 e + l.  One step of the network: each element
// meets its partner i ^ M and keeps the smaller of the two if its own bit H
// (the top bit of M) is clear.
template <int E, int M, int H>
__device__ __forceinline__ void sort_step(uint64_t v[E], int lane) {
    constexpr int ML = M & 63, ME = M >> 6;
    uint64_t o[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const uint64_t x = v[e ^ ME];
        if constexpr (ML != 0) o[e] = lane_xor<ML>(x);
        else o[e] = x;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const bool upper = H < 64 ? (lane & H) != 0 : ((64 * e) & H) != 0;
        v[e] = (o[e] < v[e]) != upper ? o[e] : v[e];  // (equal elements are the same bits)
    }
}

template <int E, int J>
__device__ __forceinline__ void sort_halve(uint64_t v[E], int lane) {
    if constexpr (J > 0) {
        sort_step<E, J, J>(v, lane);
        sort_halve<E, J / 2>(v, lane);
    }
}

// Bitonic sort, ascending, of 64 E non-negative binary64 values as bit
// patterns (which order like the values): runs of K / 2 merge by a first step
// against the mirrored partner i ^ (K - 1), then half-cleaners, so every
// comparison points the same way.
template <int E, int K = 2>
__device__ __forceinline__ void wave_sort(uint64_t v[E], int lane) {
    sort_step<E, K - 1, K / 2>(v, lane);
    sort_halve<E, K / 4>(v, lane);
    if constexpr (K < 64 * E) wave_sort<E, 2 * K>(v, lane);
}

// A row held by a wave: sample 64 e + lane in v[e], positive infinity past
// the end.
template <int E>
__device__ __forceinline__ void load_row(const double* t, int n, int lane, double v[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = 64 * e + lane < n ? t[64 * e + lane] : __builtin_inf();
}

// Whether all its n samples are valid.
template <int E>
__device__ __forceinline__ bool row_ok(const double v[E], int n, int lane) {
    bool bad = false;
#pragma unroll
    for (int e = 0; e < E; ++e) bad |= 64 * e + lane < n && !sample_ok(v[e]);
    return __builtin_amdgcn_ballot_w64(bad) == 0;
}

// Sum of a row left to right over its samples, and with BOTH of a second one
// (two independent chains).  The loop runs to a multiple of 4: adding zero
// leaves a positive sum as it is.
template <int E, bool BOTH>
__device__ __forceinline__ void row_sums(const double a[E], const double b[E], int n, int lane, double& sa, double& sb) {
    sa = 0.0;
    sb = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const bool in = 64 * e + lane < n;
        const double x = in ? a[e] : 0.0, y = BOTH && in ? b[e] : 0.0;
        const int m = min(64, n - 64 * e);
        for (int i = 0; i < m; i += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                sa = __dadd_rn(sa, readlane_f64(x, i + u));
                if constexpr (BOTH) sb = __dadd_rn(sb, readlane_f64(y, i + u));
            }
        }
    }
}

// Rows of at most 64 E samples: a work-group per candidate, a wave per row
// (striding over the shapes), then the candidate's score.  A wave also sums
// the baseline's row of its shape, beside its own for the work-group's first
// candidate, so the speedups and the score need nothing from another
// work-group and the whole of kb_rung_stats is one launch.  The kernel is a
// chain of latencies (a few thousand waves of some 500 instructions): the
// sort's steps are DPP permutations instead of LDS permutes where they stay
// inside 16 lanes, and the quantiles, the quotients and the stores of a row
// are one each, spread over the lanes.
// 1024 candidates x 3 shapes x 60 samples: rows and scores apart 7.4 + 6.2 us
// and a launch, this kernel 9.5 us; the promotion's batched loads 8.5 -> 5.9.
// With scores NULL only the rows are formed.  LOOP: a work-group takes several
// candidates (or rows alone); without it the baseline is always summed beside
// the row (its own row again where there is none).
constexpr int kFusedShapes = 4096;      // 64 KB of LDS
constexpr int kFusedWaves = 16;         // waves of a work-group at most
constexpr int kFusedCandidates = 8192;  // (see launch_rung_stats)
constexpr int kWaveSamples = 4;         // samples per lane at most

template <int E, bool LOOP>
__global__ __launch_bounds__(64 * kFusedWaves) void rung_kernel(RungParams p, const double* __restrict__ samples,
                                                                kb_sample_stats* __restrict__ rows,
                                                                kb_rung_score* __restrict__ scores) {
    extern __shared__ double s_mean[];  // [2][n_shapes]: own, baseline; NaN where the row is invalid (a sum of
                                        // positive samples never is)
    const int lane = threadIdx.x & 63;
    const int n = p.n_iter, S = p.n_shapes;
    double* const s_base = s_mean + S;
    const double nan = __builtin_nan("");
    for (int c = blockIdx.x; c < p.n_cands; c += gridDim.x) {
        const bool first = !LOOP || c == (int)blockIdx.x;
        for (int s = threadIdx.x >> 6; s < S; s += blockDim.x >> 6) {
            const size_t row = (size_t)c * S + s;
            const bool with_base = !LOOP || (first && p.base >= 0);
            double v[E], b[E];
            load_row<E>(samples + row * (size_t)n, n, lane, v);
            if (with_base)
                load_row<E>(samples + (p.base >= 0 ? (size_t)p.base * S + s : row) * (size_t)n, n, lane, b);
            const bool valid = row_ok<E>(v, n, lane);
            double sum, base_sum = 0.0;
            bool base_valid = false;
            if (with_base) {
                base_valid = row_ok<E>(b, n, lane) && p.base >= 0;
                row_sums<E, true>(v, b, n, lane, sum, base_sum);
            } else {
                row_sums<E, false>(v, v, n, lane, sum, base_sum);
            }
            uint64_t x[E];
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = __builtin_bit_cast(uint64_t, v[e]);
            wave_sort<E>(x, lane);
            // Lane w forms word w of the record: the mean (0), the quantiles
            // (1-4), their ratios to the median (5-7), the speedup (8; first the
            // baseline's mean).  The p-quantile of the sorted samples: linear
            // interpolation between the order statistics around h = (n - 1) p.
            const double q_p = lane == 1 ? 0.5 : lane == 2 || lane == 5 ? 0.9 : lane == 3 || lane == 6 ? 0.95 : 0.99;
            const double h = __dmul_rn((double)(n - 1), q_p);
            const int k = (int)floor(h);
            const int ka = min(k, n - 1), kb = min(k + 1, n - 1);
            uint64_t xa = __shfl((unsigned long long)x[0], ka & 63, 64);
            uint64_t xb = __shfl((unsigned long long)x[0], kb & 63, 64);
#pragma unroll
            for (int e = 1; e < E; ++e) {
                const uint64_t ya = __shfl((unsigned long long)x[e], ka & 63, 64);
                const uint64_t yb = __shfl((unsigned long long)x[e], kb & 63, 64);
                if (ka >> 6 == e) xa = ya;
                if (kb >> 6 == e) xb = yb;
            }
            const double fa = __builtin_bit_cast(double, xa), fb = __builtin_bit_cast(double, xb);
            double q = fa;
            if (k < n - 1) q = __dadd_rn(fa, __dmul_rn(__dsub_rn(h, (double)k), __dsub_rn(fb, fa)));
            const double q50 = readlane_f64(q, 1);
            const double num = lane == 0 ? sum : lane == 8 ? base_sum : q;
            const double quot = num / (lane == 0 || lane == 8 ? (double)n : q50);
            const double mean = readlane_f64(quot, 0);
            double base_mean = base_valid ? readlane_f64(quot, 8) : nan;
            if (!first && p.base >= 0) base_mean = s_base[s];
            double word = lane >= 1 && lane <= 4 ? q : quot;
            if (lane == 8) word = base_mean / mean;
            if (!valid) word = nan;
            if (lane == 9)
                word = __builtin_bit_cast(double, ((uint64_t)(valid ? 1u : 0u) << 32) | (uint32_t)n);
            if (lane < 10) ((double*)&rows[row])[lane] = word;
            if (lane == 0) {
                s_mean[s] = valid ? mean : nan;
                if (first) s_base[s] = base_mean;
            }
        }
        if (LOOP && scores == nullptr) continue;
        __syncthreads();
        if (threadIdx.x < 64) {
            // lane 0: the candidate, lane 1: the baseline.  Latency: the mean of
            // the row means, left to right; NaN if a row is invalid.
            const double* means = lane & 1 ? s_base : s_mean;
            double lat = 0.0;
            bool ok = true;
            for (int s = 0; s < S; ++s) {
                const double m = means[s];
                lat = __dadd_rn(lat, m);
                ok &= m == m;
            }
            lat = ok ? lat / (double)S : nan;
            const bool own_ok = __builtin_amdgcn_readlane(ok ? 1 : 0, 0) != 0;
            const double own = readlane_f64(lat, 0), base = readlane_f64(lat, 1);
            // word 1: Eq. 2, the latency term plus the one rung term gamma(r) = alpha r + beta b_r; word 2: the
            // speedup
            double word = (lane == 1 ? 1e6 : base) / (lane == 1 ? (own > 1.0 ? own : 1.0) : own);
            if (lane == 1)
                word = __dadd_rn(word, __dadd_rn(__dmul_rn(p.alpha, (double)p.rung), __dmul_rn(p.beta, p.budget)));
            if (!own_ok) word = lane == 1 ? -__builtin_inf() : nan;
            if (lane == 0) word = own;
            if (lane == 3) word = __builtin_bit_cast(double, (uint64_t)(own_ok ? 1u : 0u));
            if (lane < 4) ((double*)&scores[c])[lane] = word;
        }
        if (!LOOP || c + (int)gridDim.x >= p.n_cands) return;
        __syncthreads();
    }
}

// One work-group per row of up to kRungMaxIter samples, sorted in LDS.
__global__ __launch_bounds__(kThreads) void rows_block_kernel(const double* __restrict__ samples,
                                                               int n, int P,
                                                               kb_sample_stats* __restrict__ rows) {
    __shared__ double s[kRungMaxIter];
    __shared__ double s_sum;
    const int row = blockIdx.x;
    const double* t = samples + (size_t)row * (size_t)n;
    int bad = 0;
    for (int i = threadIdx.x; i < P; i += kThreads) {
        const double v = i < n ? t[i] : __builtin_inf();
        bad |= i < n && !sample_ok(v);
        s[i] = v;
    }
    const bool valid = __syncthreads_or(bad) == 0;
    if (!valid) {
        if (threadIdx.x == 0) write_row(&rows[row], n, false, 0.0, 0.0, 0.0, 0.0, 0.0);
        return;
    }
    if (threadIdx.x == 0) {
        // left to right; the loads are batched so that only the adds wait
        double sum = 0.0;
        int i = 0;
        for (; i + 8 <= n; i += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = s[i + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) sum = __dadd_rn(sum, v[u]);
        }
        for (; i < n; ++i) sum = __dadd_rn(sum, s[i]);
        s_sum = sum;
    }
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < P / 2; i += kThreads) {
                const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));  // j is a power of 2
                const int hi = lo + j;
                const bool ascending = (lo & k) == 0;
                const double a = s[lo], b = s[hi];
                if ((a > b) == ascending) {
                    s[lo] = b;
                    s[hi] = a;
                }
            }
            __syncthreads();
        }
    }
    if (threadIdx.x == 0) {
        auto x = [&](int i) { return s[i]; };
        write_row(&rows[row], n, true, s_sum, quantile(x, n, 0.5), quantile(x, n, 0.9),
                  quantile(x, n, 0.95), quantile(x, n, 0.99));
    }
}

// The latency of candidate c: the mean over shapes of its row means (NaN if
// a row is invalid; `valid` reports it).
__device__ __forceinline__ double latency_of(const kb_sample_stats* rows, int c, int n_shapes,
                                             bool* valid) {
    double sum = 0.0;
    bool ok = true;
    for (int s = 0; s < n_shapes; ++s) {
        const kb_sample_stats& r = rows[(size_t)c * n_shapes + s];
        ok = ok && r.valid != 0;
        sum = __dadd_rn(sum, r.mean_us);
    }
    *valid = ok;
    return ok ? sum / (double)n_shapes : __builtin_nan("");
}

__global__ __launch_bounds__(kThreads) void scores_kernel(RungParams p, kb_sample_stats* rows,
                                                           kb_rung_score* scores) {
    const int c = blockIdx.x * kThreads + threadIdx.x;
    if (c >= p.n_cands) return;
    const double nan = __builtin_nan("");
    bool ok;
    const double lat = latency_of(rows, c, p.n_shapes, &ok);
    double base_lat = nan;
    if (p.base >= 0) {
        bool base_ok;
        base_lat = latency_of(rows, p.base, p.n_shapes, &base_ok);
    }
    kb_rung_score sc;
    sc.valid = ok ? 1 : 0;
    sc.reserved = 0;
    sc.latency_us = lat;
    if (ok) {
        const double lead = 1e6 / (lat > 1.0 ? lat : 1.0);
        // Eq. 2: the latency term plus the one rung term gamma(r) = alpha r + beta b_r
        sc.score = __dadd_rn(lead, __dadd_rn(__dmul_rn(p.alpha, (double)p.rung), __dmul_rn(p.beta, p.budget)));
        sc.speedup_vs_base = base_lat / lat;
    } else {
        sc.score = -__builtin_inf();
        sc.speedup_vs_base = nan;
    }
    scores[c] = sc;
    for (int s = 0; s < p.n_shapes; ++s) {
        kb_sample_stats& r = rows[(size_t)c * p.n_shapes + s];
        const double b = p.base >= 0 ? rows[(size_t)p.base * p.n_shapes + s].mean_us : nan;
        r.speedup_vs_base = r.valid ? b / r.mean_us : nan;
    }
}

// The promotion decision D (Section 3.4): rank by score, ties to the lower
// index, and promote the first ceil(n_eligible num / den) valid non-baseline
// candidates plus a valid baseline.  Ranking is by counting: candidate i's
// rank is the number of candidates that come before it.  One wave per
// candidate: its lanes split the scan over all keys (read from L2), and a
// butterfly sums their counts; no sort or atomic is needed, the ranks are a
// permutation, and `order` is their inverse.
__device__ __forceinline__ double rank_key(const kb_rung_score& s) {
    return s.valid != 0 && s.score == s.score ? s.score : -__builtin_inf();
}

__device__ __forceinline__ int wave_sum_i32(int v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// Candidate i's counts over the keys j = lane, lane + 64, ...: those before it,
// those of them that are eligible, all eligible.  B scores per lane in flight
// (one after another, the loads' latencies were most of the kernel: 1024
// candidates 8.5 -> 5.9 us with 8; but 8 for 8 candidates 3.2, 1 for them 2.6).
template <int B>
__device__ __forceinline__ void count_before(const kb_rung_score* scores, int n, int base, int i, int lane, double ki,
                                             int& before, int& before_elig, int& n_elig) {
    for (int j0 = lane; j0 < n; j0 += 64 * B) {
        double kj[B];
        int vj[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const kb_rung_score& s = scores[min(j0 + 64 * u, n - 1)];
            kj[u] = s.score;
            vj[u] = s.valid;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int j = j0 + 64 * u;
            const bool valid = vj[u] != 0;
            const double key = valid && kj[u] == kj[u] ? kj[u] : -__builtin_inf();
            const bool elig = valid && j != base && j < n;
            const bool b = j < n && (key > ki || (key == ki && j < i));
            before += b;
            before_elig += b && elig;
            n_elig += elig;
        }
    }
}

__global__ __launch_bounds__(kThreads) void promote_kernel(const kb_rung_score* __restrict__ scores,
                                                            int n, int base, int num, int den,
                                                            int32_t* __restrict__ rank,
                                                            int32_t* __restrict__ order,
                                                            int32_t* __restrict__ promoted) {
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (i >= n) return;  // whole waves
    const double ki = rank_key(scores[i]);
    const bool valid_i = scores[i].valid != 0;
    int before = 0, before_elig = 0, n_elig = 0;
    if (n <= 64) count_before<1>(scores, n, base, i, lane, ki, before, before_elig, n_elig);
    else if (n <= 128) count_before<2>(scores, n, base, i, lane, ki, before, before_elig, n_elig);
    else count_before<8>(scores, n, base, i, lane, ki, before, before_elig, n_elig);
    before = wave_sum_i32(before);
    before_elig = wave_sum_i32(before_elig);
    n_elig = wave_sum_i32(n_elig);
    if (lane != 0) return;
    const long long keep = ((long long)n_elig * num + den - 1) / den;
    rank[i] = before;
    order[before] = i;
    int p;
    if (i == base) p = valid_i ? 1 : 0;
    else p = valid_i && before_elig < keep ? 1 : 0;
    promoted[i] = p;
}

}  // namespace

hipError_t launch_rung_promote(const kb_rung_score* scores, int n, int base, int num, int den,
                               int32_t* rank, int32_t* order, int32_t* promoted, hipStream_t stream) {
    const int per_block = kThreads / 64;
    hipLaunchKernelGGL(promote_kernel, dim3((n + per_block - 1) / per_block), dim3(kThreads), 0, stream,
                       scores, n, base, num, den, rank, order, promoted);
    return hipGetLastError();
}

// Waves per work-group of rung_kernel: one per shape if the device (8192
// waves) has room for them, at least 4, at most 16, and the rows spread evenly.
// (us: 64 candidates x 16 shapes x 60 samples 16.0 with 4 waves, 10.4 with 16;
// 5000 x 17 x 60 135 with 4, 152 with 8, 195 with 16.)
int rung_waves(const RungParams& p, int* rows_per_wave) {
    const int room = 8192 / p.n_cands;
    const int most = room < 4 ? 4 : room > kFusedWaves ? kFusedWaves : room;
    *rows_per_wave = (p.n_shapes + most - 1) / most;
    return (p.n_shapes + *rows_per_wave - 1) / *rows_per_wave;
}

hipError_t launch_rung_kernel(const RungParams& p, const double* samples, kb_sample_stats* rows,
                              kb_rung_score* scores, hipStream_t stream) {
    int per_wave;
    const int waves = rung_waves(p, &per_wave);
    // two candidates per work-group once that leaves the device full: the
    // baseline is then summed for every other candidate (8000 x 4 x 60 50 us
    // with one, 44 with two, 43 with four, 46 with eight)
    const int each = (int64_t)p.n_cands * waves >= 16384 ? 2 : 1;
    const dim3 grid((p.n_cands + each - 1) / each), block(64 * waves);
    const size_t lds = 2 * sizeof(double) * (size_t)p.n_shapes;
    const bool loop = each > 1 || scores == nullptr;
    const auto launch = [&](auto one, auto several) {
        hipLaunchKernelGGL(loop ? several : one, grid, block, lds, stream, p, samples, rows, scores);
    };
    if (p.n_iter <= 64) launch(rung_kernel<1, false>, rung_kernel<1, true>);
    else if (p.n_iter <= 128) launch(rung_kernel<2, false>, rung_kernel<2, true>);
    else launch(rung_kernel<4, false>, rung_kernel<4, true>);
    return hipGetLastError();
}

// Rows and scores in one launch, or apart.  Measured, us (candidates x shapes x
// samples; rung_kernel with the scores, rows by rung_kernel and scores_kernel,
// rows_block_kernel and scores_kernel):
//   up to 64 samples the one launch is the fastest (1 x 1 x 60 5.2, 6.7, 8.1;
//     1 x 64 x 60 33, 44, 48; 4 x 1000 x 60 486, 666, 679; 8000 x 4 x 60 44 and
//     46 before) except for very many candidates, where the scores take 64
//     lanes each in it and one lane apart (16384 x 3 x 60 67, 55; 62 before;
//     16384 x 3 x 16 37, 36; 8193 x 2 x 1 12, 16);
//   65 to 128: a row takes a wave 7 us, so few candidates with many rows per
//     wave are better spread over the device (16 x 20 x 128 21, 26, 26;
//     1 x 48 x 128 48, 37, 36; but 64 x 64 x 128 64, 72, 84);
//   129 to 256: a row takes a wave 13 us and a work-group 9 (1 x 3 x 256 15.2,
//     18.2, 12.7; 64 x 16 x 256 34, 30, 27; 64 x 64 x 256 124, 88, 96), until
//     there are candidates for most CUs (255 x 4 x 256 16.1, 20.1, 18.6;
//     1024 x 3 x 200 23, 29, 36; but 512 x 2 x 256 19.8, 20.0, 16.4).
hipError_t launch_rung_stats(const RungParams& p, const double* samples, kb_sample_stats* rows,
                             kb_rung_score* scores, hipStream_t stream) {
    const int n_rows = p.n_cands * p.n_shapes;
    int per_wave;
    rung_waves(p, &per_wave);
    const bool fits = p.n_shapes <= kFusedShapes && (p.n_cands <= kFusedCandidates || p.n_iter <= 16);
    bool fused, by_wave;  // one launch; else rows by rung_kernel
    if (p.n_iter <= 64) fused = fits, by_wave = true;
    else if (p.n_iter <= 128) fused = fits && (per_wave <= 2 || p.n_cands >= 64), by_wave = true;
    else {
        fused = fits && p.n_iter <= 64 * kWaveSamples && p.n_cands >= 192 && n_rows >= (p.n_shapes >= 3 ? 768 : 1200);
        by_wave = p.n_iter <= 64 * kWaveSamples && n_rows >= 4096;
    }
    if (fused) return launch_rung_kernel(p, samples, rows, scores, stream);
    hipError_t e;
    if (by_wave) {
        // every row a candidate of one shape without a baseline
        RungParams q = p;
        q.n_cands = n_rows;
        q.n_shapes = 1;
        q.base = -1;
        e = launch_rung_kernel(q, samples, rows, nullptr, stream);
    } else {
        int P = 1;
        while (P < p.n_iter) P <<= 1;
        hipLaunchKernelGGL(rows_block_kernel, dim3(n_rows), dim3(kThreads), 0, stream, samples, p.n_iter, P, rows);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    // (sets the rows' speedups too)
    hipLaunchKernelGGL(scores_kernel, dim3((p.n_cands + kThreads - 1) / kThreads), dim3(kThreads), 0,
                       stream, p, rows, scores);
    return hipGetLastError();
}

}  // namespace kb
