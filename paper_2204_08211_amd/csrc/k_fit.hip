// GenNorm parameters of the corrected gradient from the data, and the model code's weights from
// those parameters, without a host round trip (Sec. III eq. (kurtosis): mean, variance and
// kurtosis of GenNorm(mu, alpha, beta); Sec. IV-A (ii): the Huffman code is designed under the
// GenNorm assumption; Sec. VI: the fitted parameters are then held for several epochs).
//
//   k_moments        one read sweep over g and m: per chunk the sums of v, v^2, v^3, v^4 in fp64,
//                    v = fl32(g + fl32(gamma m)) (eq. (f_error_fb)); a wavefront owns a chunk, a
//                    lane adds its elements in index order, the wavefront folds the lanes in a
//                    fixed order: the sums do not depend on scheduling
//   k_fit_params     per (user, layer): folds the chunk sums in a fixed order, central moments,
//                    beta from the kurtosis by bisection (its steps evaluated ahead), alpha from the variance
//   k_model_weights  per code table: the element-count-weighted mixture of the quantized models
//                    of the (user, layer) pairs the table serves -> integer Huffman weights
//
// The raw-moment route loses about (mu / sigma)^4 ulps of the fourth central moment to
// cancellation; gradient layers have |mu| << sigma.
// HBM traffic of k_moments per element: read g (4) + read m (4).
#include "co3_internal.h"
#include "gennorm_math.h"

namespace co3 {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kMoWaves = 4;                 // wavefronts (chunks) per workgroup
constexpr int kMoThreads = 64 * kMoWaves;

__device__ inline uint32_t fit_find_chunk_segment(const SegDev *segs, uint32_t nseg, uint64_t chunk)
{
    uint32_t lo = 0, hi = nseg;  // segs[nseg].chunk_start = nchunks > chunk
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (segs[mid].chunk_start <= chunk) lo = mid; else hi = mid;
    }
    return lo;
}

struct Sums4 {
    double s1, s2, s3, s4;
    __device__ inline void add(float vf)
    {
        const double v = (double)vf, v2 = v * v;  // v2 is exact
        s1 += v;
        s2 += v2;
        s3 += v2 * v;
        s4 += v2 * v2;
    }
};

__global__ __launch_bounds__(kMoThreads) void k_moments(Layout lay, const float *__restrict__ g,
                                                        const float *__restrict__ m, uint64_t row_stride,
                                                        float gamma, double *__restrict__ partial)
{
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t c = (uint64_t)blockIdx.x * kMoWaves + wave;
    const uint32_t u = blockIdx.y;
    if (c >= lay.nchunks) return;  // whole wavefront; no workgroup barriers below
    const uint32_t seg = fit_find_chunk_segment(lay.segs, lay.nseg, c);
    const SegDev sd = lay.segs[seg];
    const uint64_t e0 = sd.offset + (c - sd.chunk_start) * kChunk;
    const uint64_t left = sd.offset + sd.length - e0;
    const uint32_t n = left < (uint64_t)kChunk ? (uint32_t)left : (uint32_t)kChunk;
    const float *gu = g + (uint64_t)u * row_stride + e0;
    const float *mu = m + (uint64_t)u * row_stride + e0;

    // every lane adds its elements in a fixed order: four consecutive ones at a time on the vector
    // path, every 64th element of the chunk otherwise
    Sums4 acc = {0.0, 0.0, 0.0, 0.0};
    if (n == (uint32_t)kChunk && (e0 & 3u) == 0) {
#pragma unroll 4
        for (int r = 0; r < kChunk / 4 / 64; ++r) {
            const uint32_t i = 4u * (lane + 64u * r);
            const f4 gv = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(gu + i));
            const f4 mv = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(mu + i));
#pragma unroll
            for (int j = 0; j < 4; ++j) acc.add(__fadd_rn(gv[j], __fmul_rn(gamma, mv[j])));
        }
    } else {
        for (uint32_t i = lane; i < n; i += 64) acc.add(__fadd_rn(gu[i], __fmul_rn(gamma, mu[i])));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        acc.s1 += __shfl_xor(acc.s1, o, 64);
        acc.s2 += __shfl_xor(acc.s2, o, 64);
        acc.s3 += __shfl_xor(acc.s3, o, 64);
        acc.s4 += __shfl_xor(acc.s4, o, 64);
    }
    if (lane == 0) {
        double *p = partial + ((uint64_t)u * lay.nchunks + c) * 4;
        p[0] = acc.s1; p[1] = acc.s2; p[2] = acc.s3; p[3] = acc.s4;
    }
}

// beta_of_kurtosis() by the workgroup: the same bisection, kFitDepth steps at a time.  An evaluation is three
// log-gammas, which depend on the step before, so the midpoints of the next kFitDepth steps, whichever way
// those turn out, are evaluated side by side, each log-gamma by a thread of its own: threads k, k + 256 and k + 512 take
// those of node k of the binary tree of intervals (heap order; node 0 is the range's lower end in the first round and its upper
// one in the second), and every thread then walks down the tree with the answers.  Midpoints, sums and
// decisions are the serial bisection's, bit for bit; it ends once a whole walk leaves the interval as it was, which the
// serial one's remaining steps would, too.
// Two workgroups of 768 threads fit a CU up to 80 registers, which the log-gamma takes as a function of its own (inlined, its
// constants stay in registers over the loop: 168 and spills, and one workgroup a CU).  With more pairs than CUs the
// evaluations bound it and not their chain, and a workgroup has 256 threads, thread k all three of node k.
// (One thread, 80 evaluations one after the other: k_fit_params 168 us; 256 threads 37; 768 32.  The whole fit of 8 pairs of
// 20 000 elements, 256 threads and 768: 43.8 and 38.5 us; of 256 pairs 51.4 and 46.4; 257 57.1 and 61.5; 384 63 and 67; 1200 123
// and 152; inlined, 768 threads took 58 us for 256 pairs, 90 for 384 and 198 for 1200.)
constexpr int kFitDepth = 8;
constexpr int kFitNodes = 1 << kFitDepth;
constexpr int kFitThreads = 3 * kFitNodes, kFitThreadsMany = kFitNodes;
constexpr uint64_t kFitPairsWide = 256;   // as many as CUs
struct FitGammas { double lg[3][kFitNodes]; uint8_t right[kFitNodes]; };
__device__ __attribute__((noinline)) double fit_log_gamma(uint32_t which, double b) { return lgamma((which == 0 ? 5.0 : which == 1 ? 1.0 : 3.0) / b); }
template <int kThreads>
__device__ inline double fit_beta_of_kurtosis(double kappa, uint32_t t, FitGammas *s)
{
    if (!(kappa == kappa) || isinf(kappa)) return kBetaMin;   // the same in every thread
    const double lk = log(kappa);
    const uint32_t node = t % kFitNodes;
    double lo = log(kBetaMin), hi = log(kBetaMax);
    for (int i = 0; i < 80; i += kFitDepth) {
        double at_beta = i ? kBetaMax : kBetaMin;
        if (node) {
            double a = lo, b = hi;
            for (int l = 30 - __clz((int)node); l >= 0; --l) {   // from the bit below the leading one down
                const double mid = 0.5 * (a + b);
                if ((node >> l) & 1u) a = mid; else b = mid;
            }
            at_beta = exp(0.5 * (a + b));
        }
        if (node || i <= kFitDepth) {
#pragma unroll 1
            for (uint32_t which = t / kFitNodes; which < 3u; which += kThreads / kFitNodes) s->lg[which][node] = fit_log_gamma(which, at_beta);
        }
        __syncthreads();
        if (i <= kFitDepth) {   // two rounds take place in any case
            const double end = s->lg[0][0] + s->lg[1][0] - 2.0 * s->lg[2][0];
            if (i == 0 ? lk >= end : lk <= end) return i ? kBetaMax : kBetaMin;   // the same in every thread
        }
        if (t < (uint32_t)kFitNodes && node) s->right[node] = s->lg[0][node] + s->lg[1][node] - 2.0 * s->lg[2][node] > lk;
        __syncthreads();
        const double lo0 = lo, hi0 = hi;
        uint32_t at = 1;
        for (int l = 0; l < kFitDepth; ++l) {
            const double mid = 0.5 * (lo + hi);
            const uint32_t right = s->right[at];
            if (right) lo = mid; else hi = mid;
            at = 2 * at + right;
        }
        if (lo == lo0 && hi == hi0) break;
    }
    return exp(0.5 * (lo + hi));
}

template <int kThreads>
__global__ __launch_bounds__(kThreads, kThreads == kFitThreads ? 6 : 7) void k_fit_params(Layout lay, const double *__restrict__ partial,
                                                            co3_gennorm_params *__restrict__ params)
{
    constexpr int kFold = 256;   // threads that fold the chunks' sums
    __shared__ double s_red[4][kFold];
    __shared__ FitGammas s_gammas;
    const uint32_t seg = blockIdx.x, u = blockIdx.y, t = threadIdx.x;
    const uint64_t cs = lay.segs[seg].chunk_start, ce = lay.segs[seg + 1].chunk_start;
    if (t < (uint32_t)kFold) {
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
        for (uint64_t c = cs + t; c < ce; c += kFold) {   // eight chunks' sums requested together, added in order
            const double *p = partial + ((uint64_t)u * lay.nchunks + c) * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] += p[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) s_red[j][t] = a[j];
    }
    __syncthreads();
    for (uint32_t o = kFold / 2; o > 0; o >>= 1) {   // every sum of a pair by a thread: in the first step more than the smaller workgroup has
        for (uint32_t k = t; k < 4u * o; k += kThreads) s_red[k / o][k % o] += s_red[k / o][k % o + o];
        __syncthreads();
    }
    co3_gennorm_params out = {0.0, 0.0, 0.0, 0.0};
    const uint64_t n = lay.segs[seg].length;
    if (n > 0) {   // the same in every thread, like everything below
        const double dn = (double)n;
        const double S1 = s_red[0][0], S2 = s_red[1][0], S3 = s_red[2][0], S4 = s_red[3][0];
        const double mean = S1 / dn, ms = S2 / dn;
        const double m2 = ms - mean * mean;
        const double m4 = (S4 - 4.0 * mean * S3 + 6.0 * mean * mean * S2) / dn - 3.0 * mean * mean * mean * mean;
        out.mu = mean;
        // a variance below 2^-40 of the mean square is rounding noise of the raw sums: constant layer
        if (m2 > ms * 9.094947017729282e-13) {
            out.kurtosis = m4 / (m2 * m2);
            out.beta = fit_beta_of_kurtosis<kThreads>(out.kurtosis, t, &s_gammas);
            // variance_factor(), its two log-gammas side by side
            __syncthreads();
            if (t == 0 || t == 64) s_gammas.lg[0][t / 64] = fit_log_gamma(t ? 1u : 2u, out.beta);
            __syncthreads();
            out.alpha = sqrt(m2 / exp(s_gammas.lg[0][0] - s_gammas.lg[0][1]));
        }
    }
    if (t == 0) params[(uint64_t)u * lay.nseg + seg] = out;
}

// Weights of code table b: the masses of its (user, layer) pairs are summed per symbol in the order of the pairs.  What
// bounds it is the length of one evaluation (a power and an incomplete gamma function in fp64, some microseconds),
// not their number, so an evaluation gets a thread: a workgroup takes kMwSymbols symbols and kMwPairs pairs at a time,
// two neighbouring threads the two ends of a cell.  (Thread per symbol, ends and pairs one after the other: 121
// against 15 us for eight users in [1,5,2], 1.05 ms for sixteen in [1,5,6].)
constexpr int kMwSymbols = 16;
constexpr int kMwPairs = 8;
constexpr int kMwThreads = 2 * kMwSymbols * kMwPairs;
__global__ __launch_bounds__(kMwThreads) void k_model_weights(Layout lay, const co3_gennorm_params *__restrict__ params,
                                                              uint64_t *__restrict__ weights)
{
    __shared__ uint64_t s_pair[kMwThreads];            // the pairs of a block of kMwThreads candidates that count, in order
    __shared__ uint32_t s_cnt[kMwThreads / 64];
    __shared__ double s_term[kMwPairs][kMwSymbols];
    const uint32_t b = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t end = t & 1u, sl = (t >> 1) % kMwSymbols, slot = (t >> 1) / kMwSymbols;
    const uint32_t s = blockIdx.y * kMwSymbols + sl;   // may lie beyond the alphabet (symbol_cell refuses it)
    const uint64_t first = (lay.per_user_books ? (uint64_t)(b / lay.books_per_user) : 0u) * lay.nseg;
    const uint64_t npair = lay.per_user_books ? (uint64_t)lay.nseg : (uint64_t)lay.U * lay.nseg;
    const int32_t book = (int32_t)(lay.per_user_books ? b % lay.books_per_user : b);
    double ends[2];
    const bool producible = s < lay.A && symbol_cell(s, lay.E, lay.M, lay.bias[0], &ends[0], &ends[1]);  // the same for every bias
    double mass = 0.0, count = 0.0;                    // of thread `sl`'s symbol, in the threads of slot 0
    for (uint64_t base = 0; base < npair; base += kMwThreads) {
        const uint64_t cand = first + base + t;
        bool use = base + t < npair;
        if (use) {
            const SegDev sd = lay.segs[cand % lay.nseg];
            const co3_gennorm_params p = params[cand];
            use = sd.book == book && sd.length != 0 && p.alpha > 0.0 && p.beta > 0.0;
        }
        const uint64_t mask = __ballot(use);
        if (lane == 0) s_cnt[wave] = (uint32_t)__popcll(mask);
        __syncthreads();
        uint32_t pos = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull)), n = 0;
        for (uint32_t k = 0; k < kMwThreads / 64; ++k) {
            pos += k < wave ? s_cnt[k] : 0u;
            n += s_cnt[k];
        }
        if (use) s_pair[pos] = cand;
        __syncthreads();
        for (uint32_t i0 = 0; i0 < n; i0 += kMwPairs) {
            const uint32_t i = i0 + slot;
            if (i < n) {                               // the same in both threads of a cell
                const uint64_t pr = s_pair[i];
                double F = 0.0, S = 0.0;
                if (producible) {
                    const co3_gennorm_params p = params[pr];
                    symbol_cell(s, lay.E, lay.M, lay.bias[pr], &ends[0], &ends[1]);
                    // with a real-valued scale the conversion sees y = v * gain: the model's location and scale times gain
                    const double gn = (double)lay.gain[2 * pr];
                    gennorm_cdf(ends[end], p.mu * gn, p.alpha * gn, p.beta, &F, &S);
                }
                const double Fhi = __shfl_xor(F, 1, 64), Shi = __shfl_xor(S, 1, 64);
                if (end == 0) s_term[slot][sl] = (double)lay.segs[pr % lay.nseg].length * mass_between(F, S, Fhi, Shi);
            }
            __syncthreads();
            const uint32_t nk = n - i0 < (uint32_t)kMwPairs ? n - i0 : (uint32_t)kMwPairs;
            if (slot == 0)
                for (uint32_t k = 0; k < nk; ++k) {
                    mass += s_term[k][sl];
                    count += (double)lay.segs[s_pair[i0 + k] % lay.nseg].length;
                }
            __syncthreads();
        }
    }
    if (slot == 0 && end == 0 && s < lay.A) {
        uint64_t w = 0;
        if (producible) {
            w = 1;
            if (count > 0.0) {
                const double x = floor(mass / count * 1099511627776.0);  // 2^40
                if (x >= 1.0) w = (uint64_t)x;
            }
        }
        weights[(uint64_t)b * lay.A + s] = w;
    }
}

// Exponent bias from the model, eq. (exp bias) with integer b.  The expected squared error of a candidate
// bias is a sum of non-negative shares, one per symbol's cell, so any few shares bound it from below; and
// what lies in a binade is at most half its gap away from its representative, which bounds it from above:
//   k_model_bias_bounds  per (user, layer), a workgroup per kBoundCands candidates: the shares of the zero cell and
//                        of the two outermost cells (too coarse a set loses in the first, too narrow a one in the others),
//                        and, for few pairs, from the shares of the binades the least upper bound of its candidates
//   k_model_bias_ref     for many: per (user, layer), the candidate with the smallest lower bound, evaluated in full
//   k_model_bias_errors  err_slots() workgroups per (layer, user), or one per candidate, take those whose lower bound does not
//                        exceed that (a handful of the 226; no other can be the minimum or tie with it): the
//                        integral of (x - r)^2 f(x) over every symbol's cell in closed form, folded in a fixed order -> expected
//                        squared error of the candidate
//   k_model_bias_pick    wavefront per (user, layer): the smallest bias whose error is within kBiasTie of the
//                        minimum (a format with many binades has a plateau of equally good biases;
//                        the smallest has the most headroom).  No model (alpha = 0): the IEEE bias.
// What bounds all of it is the incomplete gamma functions in fp64 (a power, an exponential, a series with a division
// per term: some microseconds each, three moments at every place where two cells meet).  Each is evaluated once, by a
// thread of its own, for both cells that meet there, the moments one after the other so that a wavefront's lanes run
// the same shape at neighbouring places; what they share, the log-gammas of the three shapes, once per workgroup.
// For few pairs that is a chain, so a workgroup has a thread for each place and moment of 256 symbols; many pairs fill
// the device and take four wavefronts (in the formats in which the search has a workgroup for
// every candidate, most only find that theirs is ruled out).  us, a thread per symbol with its six integrals one after the other / eight threads per symbol, 1024 to
// a workgroup, every place twice / this way: the bias search of 8 pairs in [1,5,2] 324 / 109 / 75, 384 pairs in
// [1,4,3] 862 / 990 / 347, 2400 pairs 4180 / 5740 / 1650, 384 pairs in [1,5,6] 8050 / 9800 / 3620; the scale search of 8 pairs in
// [1,4,3] 6190 / 3630 / 2160, 2400 pairs 33 900 / 41 500 / 15 300.
constexpr int kBiasSlots = 256;  // error slots per (user, layer); candidates: at most 226
constexpr double kBiasPrune = 1e-6;  // margin of the bound test, far above the rounding of the sums and the tie width
constexpr int kErrPlaces = kMaxA + 1;               // where the cells of a block of 256 symbols meet, and the next one's
constexpr int kErrThreads = 768;                    // 3 x 252 places for the largest alphabet of up to 8 bits
constexpr int kErrThreadsMany = kMaxA;
// Pairs from which a workgroup takes kErrThreadsMany: the candidates' search, some six of whose 226 workgroups a pair (as
// they then were) evaluated (40 pairs: 118 us with kErrThreads, 120 with kErrThreadsMany; 96 pairs: 196 and 154), and the kernels with
// one workgroup a pair, which from then on are one on every CU (the scale search of 192 pairs: 2340 and 3170 us; of
// 384: 4390 and 4070).
// Alphabets of up to 64 symbols have no more than 180 places and moments ([1,5,0]).
constexpr uint64_t kErrManySearch = 40, kErrManyOne = 256;
inline uint32_t err_threads(const Layout &lay, uint64_t many)
{
    return (uint64_t)lay.U * lay.nseg < many && lay.A > 64u ? kErrThreads : kErrThreadsMany;
}
constexpr uint64_t kUpperPairs = 64;   // pairs from which the candidates are compared with one that is evaluated first

// What the cells of one (mu, alpha, beta) share: per moment the log-gamma of its shape and the moment's factor.
struct ErrModel { double lg[3], ck[3]; };
__device__ inline void err_log_gammas(ErrModel *em, uint32_t t, double beta)
{
    if (t < 3u) em->lg[t] = lgamma(((double)t + 1.0) / beta);
    __syncthreads();
}
__device__ inline void err_factors(ErrModel *em, uint32_t t, double alpha)   // of this alpha; log-gammas are there
{
    if (t < 3u) em->ck[t] = moment_scale((int)t, alpha, em->lg[t], em->lg[0]);
    __syncthreads();
}

// P and Q of a moment at a place |x - mu|, place by place
template <int kN> struct ErrPlaces { double P[3][kN], Q[3][kN]; };

// The place where the cells of magnitude codes k and k + 1 meet, on the negative axis if neg (what symbol_cell returns)
__device__ inline double err_place(bool neg, int k, int M, int bias)
{
    const double x = 0.5 * (magnitude_of_code(k, M, bias) + magnitude_of_code(k + 1, M, bias));
    return neg ? -x : x;
}
template <int kN>
__device__ inline void err_eval(ErrPlaces<kN> *pl, uint32_t place, uint32_t k, double x, double mu, double alpha, double beta, const ErrModel *em)
{
    double P, Q;
    inc_gamma(((double)k + 1.0) / beta, pow(fabs(x - mu) / alpha, beta), em->lg[k], &P, &Q);
    pl->P[k][place] = P;
    pl->Q[k][place] = Q;
}

// sq_error_of_symbol() from the places its cell (lo, hi] ends at; at +-infinity P = 1, and where the cell reaches over
// the location its two sides start there, P = 0.
template <int kN>
__device__ inline double err_of_symbol(uint32_t s, int E, int M, int bias, double mu, const ErrPlaces<kN> *pl, uint32_t place_lo,
                                       uint32_t place_hi, const ErrModel *em)
{
    double lo, hi;
    if (!symbol_cell(s, E, M, bias, &lo, &hi)) return 0.0;
    const int code = (int)(s & ((1u << (E + M)) - 1u));
    const double r = ((s >> (E + M)) & 1u) ? -magnitude_of_code(code, M, bias) : magnitude_of_code(code, M, bias);
    const double c = r - mu, a = lo - mu, b = hi - mu;
    double j[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double pos = 0.0, neg = 0.0;
        const double Pl = isinf(lo) ? 1.0 : pl->P[k][place_lo], Ql = isinf(lo) ? 0.0 : pl->Q[k][place_lo];
        const double Ph = isinf(hi) ? 1.0 : pl->P[k][place_hi], Qh = isinf(hi) ? 0.0 : pl->Q[k][place_hi];
        if ((b > 0.0 ? b : 0.0) > (a > 0.0 ? a : 0.0)) pos = moment_between(em->ck[k], a > 0.0 ? Pl : 0.0, a > 0.0 ? Ql : 1.0, Ph, Qh);
        if ((-a > 0.0 ? -a : 0.0) > (-b > 0.0 ? -b : 0.0)) neg = moment_between(em->ck[k], -b > 0.0 ? Ph : 0.0, -b > 0.0 ? Qh : 1.0, Pl, Ql);
        j[k] = (k & 1) ? pos - neg : pos + neg;
    }
    return sq_error_of_moments(c, j[0], j[1], j[2]);
}

// Expected squared error of one candidate by a workgroup of nt >= 256 threads: the shares of symbols i, i + 256, ...
// are added in this order (one symbol for alphabets of up to 8 bits), then the 256 sums in a fixed tree.
__device__ inline double err_total(double *s_red, ErrPlaces<kErrPlaces> *pl, uint32_t t, uint32_t nt, uint32_t A, int E, int M, int bias,
                                   double mu, double alpha, double beta, const ErrModel *em)
{
    const uint32_t half = 1u << (E + M);
    const int nmag = ((1 << E) - 1) << M;      // magnitude codes Q_fp can produce: they meet at nmag - 1 places
    const bool byte = A <= (uint32_t)kMaxA;    // both signs in one block, else blocks of one sign
    double e = 0.0;
    for (uint32_t s0 = 0; s0 < A; s0 += kMaxA) {
        const bool neg0 = s0 >= half;
        const int k0 = (int)(s0 & (half - 1u));
        if (!byte && k0 >= nmag) continue;     // the same in every thread
        // byte: places 0 .. nmag - 2 on the positive axis, then the negative one's; else place i is that between
        // k0 - 1 + i and the next code, and before code 0 the zero cell's lower end
        const uint32_t n = byte ? 2u * (uint32_t)(nmag - 1) : (uint32_t)kErrPlaces;
#pragma unroll 1
        for (uint32_t i = t; i < 3u * n; i += nt) {
            const uint32_t k = (i >= n ? 1u : 0u) + (i >= 2u * n ? 1u : 0u), place = i - k * n;
            bool neg = neg0;
            int code = k0 - 1 + (int)place;
            if (byte) {
                neg = place >= (uint32_t)(nmag - 1);
                code = (int)place - (neg ? nmag - 1 : 0);
            } else if (code < 0) {
                neg = true;
                code = 0;
            }
            if (code < nmag - 1) err_eval(pl, place, k, err_place(neg, code, M, bias), mu, alpha, beta, em);
        }
        __syncthreads();
        if (t < (uint32_t)kMaxA && s0 + t < A) {
            const bool neg = byte ? t >= half : neg0;
            const int code = (int)((s0 + t) & (half - 1u));
            const uint32_t base = byte ? (neg ? (uint32_t)(nmag - 1) : 0u) : 1u;   // the place beyond code k0
            const uint32_t outer = base + (uint32_t)(code - k0);
            const uint32_t inner = byte && code == 0 ? (uint32_t)(nmag - 1) : outer - 1u;   // the zero cell's: below zero
            e += err_of_symbol(s0 + t, E, M, bias, mu, pl, neg ? outer : inner, neg ? inner : outer, em);
        }
        __syncthreads();
    }
    if (t < (uint32_t)kMaxA) s_red[t] = e;
    __syncthreads();
    for (int o = kMaxA / 2; o > 0; o >>= 1) {
        if (t < (uint32_t)o) s_red[t] += s_red[t + o];
        __syncthreads();
    }
    const double r = s_red[0];
    __syncthreads();
    return r;
}

// Places where a workgroup of the bounds' kernel evaluates: four a candidate and moment, and for the upper bounds, of the
// distribution function, the ends of all binades that its candidates' sets have, on both axes.
constexpr int kBoundCands = 16;               // candidates per workgroup, four places each ...
constexpr int kBoundPlaces = 4 * kBoundCands; // ... and a wavefront per moment
static_assert(kBoundPlaces == 64, "a wavefront per moment");
constexpr int kMaxEdges = (1 << 7) - 1 + kBoundCands;   // (exponent fields of more than seven bits have no candidates)
constexpr int kBoundThreads = 3 * kBoundPlaces + 128;   // up to five exponent bits: an evaluation each
constexpr double kProbSlack = 1e-15;          // of differences of the distribution function
template <bool kUppers>
__global__ __launch_bounds__(kUppers ? kBoundThreads : 3 * kBoundPlaces) void k_model_bias_bounds(
    Layout lay, const co3_gennorm_params *__restrict__ params, double *__restrict__ bounds)
{
    __shared__ ErrModel s_em;
    __shared__ ErrPlaces<kBoundPlaces> s_pl;
    __shared__ double s_share[kBoundCands][3];
    __shared__ double s_F[2][kUppers ? kMaxEdges : 1];      // distribution function at -2^e and 2^e
    __shared__ double s_upper[kBoundCands];
    const uint32_t seg = blockIdx.y, u = blockIdx.z, t = threadIdx.x;
    const uint32_t cand0 = blockIdx.x * kBoundCands;
    const uint64_t pair = (uint64_t)u * lay.nseg + seg;
    const co3_gennorm_params p = params[pair];
    const uint32_t ncand = (uint32_t)(kBiasMax - bias_min_supported(lay.E) + 1);
    const int bias0 = bias_min_supported(lay.E) + (int)cand0;
    const bool model = p.alpha > 0.0 && p.beta > 0.0;   // the same in every thread
    const uint32_t binades = (1u << lay.E) - 2u, edges = binades + kBoundCands;
    const int edge0 = 1 - (bias0 + kBoundCands - 1);    // exponent of the lowest edge
    if (model) {
        err_log_gammas(&s_em, t, p.beta);
        err_factors(&s_em, t, p.alpha);
        const uint32_t top = (((1u << lay.E) - 1u) << lay.M) - 1u;        // largest magnitude code
        if constexpr (!kUppers) {
            const uint32_t place = t % kBoundPlaces, which = place & 3u;      // above and below zero, before the outermost cells
            if (cand0 + (place >> 2) < ncand)
                err_eval(&s_pl, place, t / kBoundPlaces, err_place((which & 1u) != 0u, (which & 2u) ? (int)top - 1 : 0, lay.M, bias0 + (int)(place >> 2)),
                         p.mu, p.alpha, p.beta, &s_em);
        } else {
#pragma unroll 1
            for (uint32_t job = t; job < 3u * kBoundPlaces + 2u * edges; job += kBoundThreads) {
                const bool cell = job < 3u * kBoundPlaces;
                const uint32_t place = job % kBoundPlaces, which = place & 3u;    // above and below zero, before the outermost cells
                const uint32_t edge = (job - 3u * kBoundPlaces) >> 1, plus = (job - 3u * kBoundPlaces) & 1u;
                if (cell && cand0 + (place >> 2) >= ncand) continue;
                const uint32_t k = cell ? job / kBoundPlaces : 0u;
                const double x = cell ? err_place((which & 1u) != 0u, (which & 2u) ? (int)top - 1 : 0, lay.M, bias0 + (int)(place >> 2))
                                      : (plus ? ldexp(1.0, edge0 + (int)edge) : -ldexp(1.0, edge0 + (int)edge));
                double P, Q;
                inc_gamma(((double)k + 1.0) / p.beta, pow(fabs(x - p.mu) / p.alpha, p.beta), s_em.lg[k], &P, &Q);
                if (cell) {
                    s_pl.P[k][place] = P;
                    s_pl.Q[k][place] = Q;
                } else {
                    s_F[plus][edge] = x >= p.mu ? 0.5 + 0.5 * P : 0.5 * Q;
                }
            }
        }
        __syncthreads();
        if (t < 3u * kBoundCands && cand0 + t / 3u < ncand) {
            const uint32_t cl = t / 3u, w = t % 3u, pc = 4u * cl;
            const uint32_t sy = w == 0u ? 0u : w == 1u ? top : (1u << (lay.E + lay.M)) | top;
            s_share[cl][w] = err_of_symbol(sy, lay.E, lay.M, bias0 + (int)cl, p.mu, &s_pl, w == 0u ? pc + 1u : pc + 2u, w == 0u ? pc : pc + 3u, &s_em);
        }
        __syncthreads();
    }
    if (t < (uint32_t)kBoundCands) {
        double lower = INFINITY, upper = INFINITY;
        if (model && cand0 + t < ncand) {
            lower = s_share[t][0] + s_share[t][1] + s_share[t][2];
        }
        if (kUppers && model && cand0 + t < ncand) {
            // an element lies at most half a gap from its representative, but for those in the outermost cells
            upper = s_share[t][1] + s_share[t][2];
            const uint32_t e0 = (uint32_t)(kBoundCands - 1) - t;             // the edge 2^(1 - bias)
            double half_gap = ldexp(0.5, 1 - (bias0 + (int)t) - lay.M), below = 0.0;
            for (uint32_t f = 0; f <= binades; ++f) {
                const double inside = s_F[1][e0 + f] - s_F[0][e0 + f];
                upper += half_gap * half_gap * (inside - below + kProbSlack);
                below = inside;
                if (f) half_gap *= 2.0;
            }
        }
        if (cand0 + t < ncand) bounds[pair * kBiasSlots + cand0 + t] = lower;
        s_upper[t] = upper;
    }
    __syncthreads();
    if (kUppers && t == 0) {   // behind the candidates' slots
        double least = INFINITY;
#pragma unroll
        for (int i = 0; i < kBoundCands; ++i) least = s_upper[i] < least ? s_upper[i] : least;
        bounds[pair * kBiasSlots + kBiasSlots - 1 - blockIdx.x] = least;
    }
}

__global__ __launch_bounds__(kErrThreads) void k_model_bias_ref(Layout lay, const co3_gennorm_params *__restrict__ params,
                                                                const double *__restrict__ bounds, double *__restrict__ ref)
{
    __shared__ double s_red[kMaxA];
    __shared__ ErrPlaces<kErrPlaces> s_pl;
    __shared__ ErrModel s_em;
    __shared__ int s_c0;
    const uint32_t seg = blockIdx.x, u = blockIdx.y, t = threadIdx.x;
    const uint64_t pair = (uint64_t)u * lay.nseg + seg;
    const co3_gennorm_params p = params[pair];
    if (!(p.alpha > 0.0 && p.beta > 0.0)) {   // the same in every thread
        if (t == 0) ref[pair] = INFINITY;
        return;
    }
    const int ncand = kBiasMax - bias_min_supported(lay.E) + 1;
    if (t < 64u) {   // first candidate with the smallest bound
        const double *lb = bounds + pair * kBiasSlots;
        int c0 = 0;
        double v0 = lb[0];
        for (int c = (int)t; c < ncand; c += 64) {
            if (lb[c] < v0) { v0 = lb[c]; c0 = c; }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double v = __shfl_xor(v0, o, 64);
            const int c = __shfl_xor(c0, o, 64);
            if (v < v0 || (v == v0 && c < c0)) { v0 = v; c0 = c; }
        }
        if (t == 0) s_c0 = c0;
    }
    err_log_gammas(&s_em, t, p.beta);
    err_factors(&s_em, t, p.alpha);
    const double total = err_total(s_red, &s_pl, t, blockDim.x, lay.A, lay.E, lay.M, bias_min_supported(lay.E) + s_c0, p.mu, p.alpha, p.beta, &s_em);
    if (t == 0) ref[pair] = total;
}

// The candidates that are left of a pair, taken by the workgroups of the pair: kEach, one for each of all candidates, which leaves at
// once where that is ruled out, or err_slots() that share those left.  ref: the error of one, or nullptr and the least upper bounds say it.
// As many as a plateau of equally good biases is long, a binade each, and some.  (Not a multiple of eight: the first few, which find
// candidates, would all lie on the same dies: 384 pairs in [1,4,3] 494 us, 245 so.)  Where the plateau is half of the candidates, or a
// quarter with many pairs, what a workgroup does to find its own costs more than the workgroups that leave, and the loop over
// them registers (99, four wavefronts a SIMD, and 96, five).  Bias search with 61 that
// share and with one each, us: [1,7,0] 1 pair 55 and 38, 32 pairs 237 and 213, 384 pairs 1241 and 1239; [1,7,4] 32 pairs 1479 and 1281,
// 96 pairs 2905 and 2613; [1,6,1] 32 pairs 163 and 174, 63 187 and 196, 64 197 and 197, 384 906 and 872.
inline uint32_t err_slots(int E) { return E < 6 ? (1u << E) + 5u : 61u; }
inline bool err_each(int E, uint64_t pairs) { return E > 6 || (E == 6 && pairs >= kUpperPairs); }
template <bool kEach>
__global__ __launch_bounds__(kErrThreads) void k_model_bias_errors(Layout lay, const co3_gennorm_params *__restrict__ params,
                                                                   const double *__restrict__ bounds, uint32_t nbounds,
                                                                   const double *__restrict__ ref, double *__restrict__ errors)
{
    __shared__ double s_red[kMaxA];
    __shared__ ErrPlaces<kErrPlaces> s_pl;
    __shared__ ErrModel s_em;
    const uint32_t seg = blockIdx.y, u = blockIdx.z, t = threadIdx.x, lane = t & 63u;
    const uint64_t pair = (uint64_t)u * lay.nseg + seg;
    const co3_gennorm_params p = params[pair];
    const bool model = p.alpha > 0.0 && p.beta > 0.0;
    const uint32_t ncand = (uint32_t)(kBiasMax - bias_min_supported(lay.E) + 1);
    const double *lb = bounds + pair * kBiasSlots;
    const uint32_t of = kEach ? blockIdx.x : t;   // the candidate that is compared here
    const double mine = of < ncand ? lb[of] : INFINITY;
    double limit = INFINITY;
    if (ref) {
        limit = ref[pair];
    } else {
        for (uint32_t i = 0; i < nbounds; ++i) {
            const double x = lb[kBiasSlots - 1 - i];
            limit = x < limit ? x : limit;
        }
    }
    // a candidate whose lower bound lies above another's error, or upper bound, cannot win or tie
    const bool left = model && of < ncand && !(mine > limit * (1.0 + kBiasPrune));
    auto evaluate = [&](uint32_t cand) {
        const double total = err_total(s_red, &s_pl, t, blockDim.x, lay.A, lay.E, lay.M, bias_min_supported(lay.E) + (int)cand, p.mu, p.alpha, p.beta, &s_em);
        if (t == 0) errors[pair * kBiasSlots + cand] = total;
    };
    if constexpr (kEach) {
        if (!left) {   // the same in every thread
            if (t == 0) errors[pair * kBiasSlots + of] = INFINITY;
            return;
        }
        err_log_gammas(&s_em, t, p.beta);
        err_factors(&s_em, t, p.alpha);
        evaluate(of);
    } else {
        __shared__ uint8_t s_left[kBiasSlots];
        __shared__ uint32_t s_count[kBiasSlots / 64];
        const uint64_t mask = __ballot(left);
        if (lane == 0 && t < (uint32_t)kBiasSlots) s_count[t >> 6] = (uint32_t)__popcll(mask);
        if (blockIdx.x == 0 && t < ncand && !left) errors[pair * kBiasSlots + t] = INFINITY;
        __syncthreads();
        uint32_t n = 0, rank = (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        for (uint32_t k = 0; k < (uint32_t)kBiasSlots / 64u; ++k) {
            rank += k < (t >> 6) ? s_count[k] : 0u;
            n += s_count[k];
        }
        if (left) s_left[rank] = (uint8_t)t;
        if (blockIdx.x >= n) return;   // the same in every thread
        err_log_gammas(&s_em, t, p.beta);
        err_factors(&s_em, t, p.alpha);
        for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) evaluate(s_left[i]);
    }
}

__global__ __launch_bounds__(64) void k_model_bias_pick(Layout lay, const double *__restrict__ errors,
                                                        int32_t *__restrict__ bias_out, double *__restrict__ error_out)
{
    const uint64_t i = blockIdx.x;  // (user, layer) pair
    const double *err = errors + i * kBiasSlots;
    const int b0 = bias_min_supported(lay.E);
    const int ncand = kBiasMax - b0 + 1;
    const int lane = (int)threadIdx.x;
    constexpr int kPer = kBiasSlots / 64;
    double e[kPer], lowest = INFINITY;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int c = lane + 64 * r;
        e[r] = c < ncand ? err[c] : INFINITY;
        lowest = e[r] < lowest ? e[r] : lowest;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double v = __shfl_xor(lowest, o, 64);
        lowest = v < lowest ? v : lowest;
    }
    int best = (1 << (lay.E - 1)) - 1;
    double best_err = 0.0;
    if (lowest < INFINITY) {
        const double limit = lowest * (1.0 + kBiasTie);
        int first = ncand;          // the first candidate within the limit; there is one, the lowest itself
        double first_err = 0.0;
#pragma unroll
        for (int r = kPer - 1; r >= 0; --r) {
            if (e[r] <= limit) { first = lane + 64 * r; first_err = e[r]; }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const int c = __shfl_xor(first, o, 64);
            const double v = __shfl_xor(first_err, o, 64);
            if (c < first) { first = c; first_err = v; }
        }
        best = b0 + first;
        best_err = first_err;
    }
    if (lane == 0) {
        bias_out[i] = best;
        if (error_out) error_out[i] = best_err;
    }
}

// errors and bounds per candidate, reference error per pair
size_t bias_workspace_bytes(const Layout &lay) { return (size_t)lay.U * lay.nseg * (2 * kBiasSlots + 1) * sizeof(double) + 256; }

hipError_t launch_model_bias(const Layout &lay, const co3_gennorm_params *params, int32_t *bias, double *error,
                             double *errors_ws, hipStream_t s)
{
    if (lay.U == 0) return hipSuccess;
    const int ncand = kBiasMax - bias_min_supported(lay.E) + 1;
    ProfScope prof(K_MODEL_BIAS, s);
    const uint64_t pairs = (uint64_t)lay.U * lay.nseg;
    double *bounds = errors_ws + pairs * kBiasSlots;
    const uint32_t nbounds = (uint32_t)(ncand + kBoundCands - 1) / kBoundCands;
    static_assert(kBiasSlots - (226 + kBoundCands - 1) / kBoundCands >= 226, "a slot for every workgroup's least upper bound behind the candidates'");
    // Few pairs wait for a chain of kernels, many for their evaluations, which one candidate's error rules out more of than an
    // upper bound does.  Bias search in [1,4,3] and [1,5,2], us: 8 pairs by an error 64 and 69, by upper bounds 46 and 46; 48 pairs 105
    // and 134, 75 and 107; 96 pairs 119 and 178, 173 and 178; 384 pairs 305 and 536, 587 and 575.
    const bool uppers = pairs < kUpperPairs;
    double *ref = uppers ? nullptr : bounds + pairs * kBiasSlots;
    if (uppers) {
        hipLaunchKernelGGL(k_model_bias_bounds<true>, dim3(nbounds, lay.nseg, lay.U), dim3(kBoundThreads), 0, s, lay, params, bounds);
    } else {
        hipLaunchKernelGGL(k_model_bias_bounds<false>, dim3(nbounds, lay.nseg, lay.U), dim3(3 * kBoundPlaces), 0, s, lay, params, bounds);
        hipLaunchKernelGGL(k_model_bias_ref, dim3(lay.nseg, lay.U), dim3(err_threads(lay, kErrManyOne)), 0, s, lay, params, bounds, ref);
    }
    const bool each = err_each(lay.E, pairs);
    hipLaunchKernelGGL(each ? k_model_bias_errors<true> : k_model_bias_errors<false>, dim3(each ? (uint32_t)ncand : err_slots(lay.E), lay.nseg, lay.U),
                       dim3(err_threads(lay, kErrManySearch)), 0, s, lay, params, bounds, nbounds, ref, errors_ws);
    hipLaunchKernelGGL(k_model_bias_pick, dim3((uint32_t)pairs), dim3(64), 0, s, lay, errors_ws, bias,
                       error);
    return hipGetLastError();
}

// eq. (exp bias) with b over the reals, per (user, layer), from the integer optimum found above.  A scale c = 2^t
// on top of an integer bias turns the representative set into {c x}; its error on GenNorm(mu, alpha, beta) is c^2
// times the error of the unscaled set on GenNorm(mu / c, alpha / c, beta), so the sum over the symbols' cells
// serves again.  The logarithm s = t - bias of the whole scale is scanned in steps of 1/16 binade over one and a
// half binades to either side of the integer optimum and refined by a golden-section search between the scan
// points next to the best one; bias = -round(s), t = s + bias in [-1/2, 1/2].  One workgroup per (user, layer),
// every evaluation folded in the same fixed order: all threads see the same numbers and take
// the same steps.  A real scale is taken only where it lowers the error by more than kBiasTie (relative).
__global__ __launch_bounds__(kErrThreads) void k_model_scale(Layout lay, const co3_gennorm_params *__restrict__ params,
                                                       int32_t *bias_io, const double *__restrict__ err_int,
                                                       float *__restrict__ gain_pairs, double *error_out)
{
    __shared__ double s_red[kMaxA];
    __shared__ ErrPlaces<kErrPlaces> s_pl;
    __shared__ ErrModel s_em;
    const uint32_t seg = blockIdx.x, u = blockIdx.y, t = threadIdx.x;
    const uint64_t pair = (uint64_t)u * lay.nseg + seg;
    const co3_gennorm_params p = params[pair];
    const int b_int = bias_io[pair];
    const double e_int = err_int[pair];
    int b_out = b_int;
    float gn = 1.0f, ig = 1.0f;
    double e_out = e_int;
    __syncthreads();   // every thread has read the integer result before thread 0 replaces it
    if (p.alpha > 0.0 && p.beta > 0.0) {   // the same in every thread
        const int bmin = bias_min_supported(lay.E), bmax = kBiasMax;
        err_log_gammas(&s_em, t, p.beta);
        // Evaluation i of the expected error: 0 .. 2 kHalf the scan, from kGold on the golden-section search (two points,
        // kSteps more, the middle of what is left), kLast that of the fp32 pair that is returned.  One loop, so that
        // the evaluation is in the code once (called from eight places it spilt 356 bytes a thread).
        constexpr int kHalf = 24, kSteps = 60, kGold = 2 * kHalf + 1, kMid = kGold + 2 + kSteps, kLast = kMid + 1;
        const double r = 0.6180339887498949, s0 = -(double)b_int;
        double best_s = s0, best_f = e_int, a = 0.0, b = 0.0, x1 = 0.0, x2 = 0.0, f1 = 0.0, f2 = 0.0;
        int best_k = 0;
#pragma unroll 1
        for (int i = 0; i <= kLast; ++i) {
            double sc;
            bool first = true;          // golden section: whether x1 is evaluated, or x2
            if (i == kGold) {
                if (best_k == -kHalf || best_k == kHalf) i = kLast;
                a = best_s - 1.0 / 16.0; b = best_s + 1.0 / 16.0;
                x1 = b - r * (b - a); x2 = a + r * (b - a);
            }
            if (i < kGold) {
                sc = s0 + (double)(i - kHalf) / 16.0;
            } else if (i < kMid) {
                first = i == kGold || (i > kGold + 1 && f1 < f2);
                if (i > kGold + 1) {
                    if (first) { b = x2; x2 = x1; f2 = f1; x1 = b - r * (b - a); }
                    else { a = x1; x1 = x2; f1 = f2; x2 = a + r * (b - a); }
                }
                sc = first ? x1 : x2;
            } else {
                sc = i == kMid ? 0.5 * (a + b) : best_s;
            }
            int eb = (int)lround(-sc);
            eb = eb < bmin ? bmin : (eb > bmax ? bmax : eb);
            double tt = sc + (double)eb;
            if (i == kLast) {
                if (!(best_f < e_int * (1.0 - kBiasTie))) break;
                ig = (float)exp2(tt);
                gn = 1.0f / ig;
                b_out = eb;
                tt = log2((double)ig);
            }
            const double c = exp2(tt);
            err_factors(&s_em, t, p.alpha / c);
            const double v = c * c * err_total(s_red, &s_pl, t, blockDim.x, lay.A, lay.E, lay.M, eb, p.mu / c, p.alpha / c, p.beta, &s_em);
            if (i < kGold) {
                if (v < best_f) { best_f = v; best_s = sc; best_k = i - kHalf; }
            } else if (i < kMid) {
                if (first) f1 = v; else f2 = v;
            } else if (i == kMid) {
                if (v < best_f) { best_f = v; best_s = sc; }
            } else {
                e_out = v;
            }
        }
    }
    if (t == 0) {
        bias_io[pair] = b_out;
        gain_pairs[2 * pair] = gn;
        gain_pairs[2 * pair + 1] = ig;
        if (error_out) error_out[pair] = e_out;
    }
}

// the integer search's workspace and its expected errors per pair
size_t scale_workspace_bytes(const Layout &lay) { return bias_workspace_bytes(lay) + (size_t)lay.U * lay.nseg * sizeof(double) + 256; }

hipError_t launch_model_scale(const Layout &lay, const co3_gennorm_params *params, int32_t *bias, float *gain_pairs,
                              double *error, double *ws, hipStream_t s)
{
    if (lay.U == 0 || lay.nseg == 0) return hipSuccess;
    const uint64_t pairs = (uint64_t)lay.U * lay.nseg;
    double *err_int = ws;   // [pairs], then the integer search's own workspace (256-byte aligned again)
    double *ws_int = reinterpret_cast<double *>((reinterpret_cast<uintptr_t>(ws + pairs) + 255u) & ~(uintptr_t)255u);
    hipError_t e = launch_model_bias(lay, params, bias, err_int, ws_int, s);
    if (e != hipSuccess) return e;
    ProfScope prof(K_MODEL_BIAS, s);
    hipLaunchKernelGGL(k_model_scale, dim3(lay.nseg, lay.U), dim3(err_threads(lay, kErrManyOne)), 0, s, lay, params, bias, err_int, gain_pairs,
                       error);
    return hipGetLastError();
}

size_t fit_workspace_bytes(const Layout &lay) { return (size_t)lay.U * lay.nchunks * 4 * sizeof(double) + 256; }

hipError_t launch_fit(const Layout &lay, const float *g, const float *m, uint64_t row_stride, float gamma,
                      co3_gennorm_params *params, double *partial, hipStream_t s)
{
    if (lay.U == 0) return hipSuccess;
    if (lay.nchunks) {
        ProfScope prof(K_MOMENTS, s);
        const uint32_t gx = (uint32_t)((lay.nchunks + kMoWaves - 1) / kMoWaves);
        hipLaunchKernelGGL(k_moments, dim3(gx, lay.U), dim3(kMoThreads), 0, s, lay, g, m, row_stride, gamma, partial);
    }
    ProfScope prof(K_FIT, s);
    if ((uint64_t)lay.U * lay.nseg <= kFitPairsWide) hipLaunchKernelGGL(k_fit_params<kFitThreads>, dim3(lay.nseg, lay.U), dim3(kFitThreads), 0, s, lay, partial, params);
    else hipLaunchKernelGGL(k_fit_params<kFitThreadsMany>, dim3(lay.nseg, lay.U), dim3(kFitThreadsMany), 0, s, lay, partial, params);
    return hipGetLastError();
}

hipError_t launch_model_weights(const Layout &lay, const co3_gennorm_params *params, uint64_t *weights,
                                hipStream_t s)
{
    if (lay.nbooks == 0) return hipSuccess;
    ProfScope prof(K_MODEL_WEIGHTS, s);
    hipLaunchKernelGGL(k_model_weights, dim3(lay.nbooks, (lay.A + kMwSymbols - 1) / kMwSymbols), dim3(kMwThreads), 0, s,
                       lay, params, weights);
    return hipGetLastError();
}

}  // namespace co3
