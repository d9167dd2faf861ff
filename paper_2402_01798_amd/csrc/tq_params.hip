// tq_params: parameter design of the truncated quantizer (arXiv 2402.01798, Sec. IV) from
// the per-bucket statistics, one workgroup per bucket; results in fp64, rounded once.
//
//   tail index      gamma = 1 + n_tail / sum ln(|g|/g_min)            (Sec. V, MLE)
//   tail mass       rho   = n_tail / (2 n)                            (one-sided, Sec. IV-A)
//   threshold       alpha = g_min [2 rho s^2 / ((gamma-2) Q(alpha))]^(1/(gamma-1)),
//                   Q = Q_U (Sec. IV-A, boxed) or Q_N (Sec. IV-B, second boxed equation)
//   codebook        uniform: l_k = -alpha + k 2alpha/s; non-uniform: the points where the
//                   integral of lambda_s ~ p^(1/3) (Sec. IV-B, first boxed equation) reaches k
//   BiScaled        (appendix "Truncated BiScaled Quantization") Q = min_k Q_B(alpha, k),
//                   Q_B = [(2 int_{k alpha}^{alpha} p)^(1/3) (1-k)^(2/3) + (2 int_0^{k alpha} p)^(1/3) k^(2/3)]^3,
//                   k over 0 and the bin edges below alpha; s_beta = the odd integer nearest to
//                   s p1^(1/3) k / (p2^(1/3) (1-k) + p1^(1/3) k) uniform cells on [-k alpha, k alpha],
//                   the other s - s_beta on the rest of [-alpha, alpha]
//
// The density p on [-alpha, alpha] is the histogram's (constant inside a bin).  With the counts
// below each bin and H[i] = int_0^{lo_i} p^(1/3), both Q_U(alpha) and the integral of p^(1/3)
// up to alpha cost O(1) per evaluation.
//
// What bounds it: latency.  A record is 3.6 KB of input and a chain of dependent scalar steps; one
// tensor's record occupies one compute unit, and even 2736 records of small buckets are only two or
// three workgroups' worth of time each.  So everything here shortens the chain:
//   - per-bin work on all lanes, bin = 256 k + lane, with wavefronts whose bins are empty skipping
//     it; scans by cross-lane moves (DPP); the cube root of an integer count
//     from the hardware's fp32 exp2/log2 and two fp64 Newton steps (the bins' widths are powers of
//     two, so nothing else needs a root), the binned tail's logarithms from a 16-entry table;
//   - the fixed point is first approached in fp32 (one iteration about 250 cycles instead of 1600),
//     by the boxed map itself and, once that provably contracts, by Newton steps on it, and
//     then polished by fp64 Newton steps on the logarithmic residual.  When the map does not
//     contract safely (see kCertifiedSlope), the plain fp64 iteration of the definition runs,
//     because there the result is where that iteration stops, not a fixed point;
//   - BiScaled's search, taken a dozen times a record, looks at the 128 edges below the threshold, a lane each, and
//     at more only if one of those could win;
//   - a lane per level for the codebook and its reciprocal widths;
//   - one kernel per codebook family: what a family does not need costs it no LDS and no
//     instruction fetch.
// Measured on MI355X, us for one launch, against all-fp64 iteration on lane 0 of one kernel for
// all families: uniform, 4 records 11.2 -> 4.7, 952 records 30.3 -> 7.2; non-uniform, 1 record
// 18.7 -> 7.7, 768 records 34.3 -> 10.4, 2736 records 78 -> 21.5; BiScaled, 391 records 128 -> 19.3.
// The search of BiScaled by one wavefront over the edges that can win instead of four over all of them, with their barriers:
// 1 record 15.9 -> 13.6, 391 19.0 -> 16.6, 952 25.6 -> 17.4, 2736 168 -> 122.
// 512 or 1024 threads per record instead of 256 gain 0.4 us on a single non-uniform record and lose
// 6 and 18 us on 2736 of them.
#include <type_traits>

#include "tq_device.h"

namespace tq {

constexpr int kNB = TQ_NBINS;
constexpr int kParamsBlock = 256;                         // threads per workgroup
constexpr int kParamsWaves = kParamsBlock / 64;
constexpr int kBinsPerLane = 1024 / kParamsBlock;         // 1024 >= 898 bins
constexpr double kGammaFloor = 2.02;
constexpr double kAlphaFloor = 5.421010862427522e-20;     // 2^-64
constexpr int kMaxIter = 100;
constexpr double kRelTol = 1e-10;
constexpr double kLn2 = 0.69314718055994530942;

constexpr double kFirstEdge = 9.094947017729282e-13;      // 2^-40, the lower edge of bin 1
__device__ __forceinline__ double bin_lo(int i)
{
    if (i <= 0) return 0.0;
    if (i >= kNB - 1) return 65536.0;
    const int j = i - 1;
    return ldexp(1.0 + (double)(j & 15) * 0.0625, (j >> 4) - 40);
}

__device__ __forceinline__ double last_bin_width(double absmax)
{
    return (absmax > 131072.0 ? absmax : 131072.0) - 65536.0;
}

// Bin whose [lo, hi) holds x >= 0 (the last bin is closed above): biased exponent and top four
// mantissa bits, as the statistics kernel bins them.
__device__ __forceinline__ int bin_of(double x)
{
    const int i = (__double2hiint(x) >> 16) - (((1023 - 40) << 4) - 1);
    return i < 0 ? 0 : (i > kNB - 1 ? kNB - 1 : i);
}

// 1 / x to about an ulp: hardware seed, two Newton steps.
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// ln x for finite x > 0: x = 2^e m with m in [sqrt(1/2), sqrt(2)), ln m = 2 artanh((m - 1) / (m + 1)), whose
// series in z = ((m - 1) / (m + 1))^2 <= 0.0295 is cut after z^10 (below 1e-17).  Evaluated in pairs
// of terms: a third of the dependent steps of the library's ln, in a third of its code.
__device__ __forceinline__ double ln(double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);             // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.70710678118654752440;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double den = m + 1.0;
    const double r = recip(den);
    double t = (m - 1.0) * r;
    t = __builtin_fma(__builtin_fma(-den, t, m - 1.0), r, t);
    const double z = t * t, z2 = z * z, z4 = z2 * z2;
    const double p01 = __builtin_fma(z, 2.0 / 5.0, 2.0 / 3.0), p23 = __builtin_fma(z, 2.0 / 9.0, 2.0 / 7.0);
    const double p45 = __builtin_fma(z, 2.0 / 13.0, 2.0 / 11.0), p67 = __builtin_fma(z, 2.0 / 17.0, 2.0 / 15.0);
    const double p89 = __builtin_fma(z, 2.0 / 21.0, 2.0 / 19.0);
    const double p03 = __builtin_fma(z2, p23, p01), p47 = __builtin_fma(z2, p67, p45);
    const double p = __builtin_fma(z4, __builtin_fma(z4, p89, p47), p03);
    return __builtin_fma((double)e, kLn2, __builtin_fma(t * z, p, t + t));
}

// log2, exp2 and the reciprocal as the hardware computes them (about 1 ulp of binary32).
__device__ __forceinline__ float log2_hw(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float rcp_hw(float x) { return __builtin_amdgcn_rcpf(x); }

// exp(x) for |x| < 170 from its own logarithm: y from the hardware's exp2, then y exp(r), r = x / 2 - ln y, |r| < 1e-4, by
// four terms, squared.  Without the library's constants the code that seldom runs leaves the rest its registers.
__device__ __forceinline__ double exp_by_ln(double x)
{
    const double y = (double)exp2_hw((float)(x * (0.5 / kLn2)));
    const double r = __builtin_fma(0.5, x, -ln(y));
    const double root = __builtin_fma(y, r * (1.0 + r * (0.5 + r * (1.0 / 6.0))), y);
    return root * root;
}

// Cube root of x >= 0: fp32 seed, two Newton steps in fp64 (the reciprocal of the derivative is
// needed to the seed's precision only); below the range of binary32 the library's.
__device__ __forceinline__ double cube_root(double x)
{
    const float xf = (float)x;
    if (xf < 1.0e-37f && x > 0.0) return cbrt(x);
    const float y0 = exp2_hw(log2_hw(xf) * (1.0f / 3.0f));
    const double r = (double)rcp_hw(3.0f * y0 * y0);
    double y = (double)y0;
    y += (x - y * y * y) * r;
    y += (x - y * y * y) * r;
    return x > 0.0 ? y : 0.0;
}

// ln((1 + m/16)(1 + (m+1)/16)) / 2: the logarithm of a bin's geometric centre within its octave,
// and ln(1 + m/16): that of its lower edge.
struct OctaveLogs { double centre[16], edge[16]; };
__constant__ OctaveLogs kOctaveLogs = {
    {0.03031231090821742, 0.089203828736409141, 0.14481664629152136, 0.1974969041204345,
     0.24753863339892576, 0.29519372330108817, 0.3406796124039515, 0.38418530089876646,
     0.42587610536829196, 0.46589745920506015, 0.50437797977312426, 0.54143196584998532,
     0.57716144784105772, 0.61165788358453343, 0.6450035708338695, 0.67727283140265515},
    {0.0, 0.06062462181643484, 0.11778303565638346, 0.17185025692665923,
     0.22314355131420976, 0.27193371548364176, 0.31845373111853459, 0.36290549368936847,
     0.40546510810816438, 0.44628710262841953, 0.48550781578170077, 0.52324814376454787,
     0.55961578793542266, 0.59470710774669278, 0.62860865942237409, 0.66139848224536502}
};

// Count of a bin and of all bins below it, exact.  Every bucket has n < 2^32; WIDE is for records that a caller
// has summed beyond that (their bins are 32-bit still): the fp64 sums for every record cost 0.5 to 1.9 us a launch, the test for such a record 0.2 to 0.4.
template <bool WIDE> struct BinCounts;
template <> struct BinCounts<false> {
    uint2 hc[kNB];
    struct Bin { uint32_t here, below; };
    __device__ __forceinline__ Bin at(int i) const { const uint2 v = hc[i]; return {v.x, v.y}; }
};
template <> struct BinCounts<true> {
    double cum[kNB + 1];
    struct Bin { double here, below; };
    __device__ __forceinline__ Bin at(int i) const { const double b = cum[i]; return {cum[i + 1] - b, b}; }
};

template <bool ROOTS, bool WIDE, bool SEARCH>
struct ParamsLds {
    BinCounts<WIDE> bins;
    double H[ROOTS ? kNB + 1 : 1];         // H[i] = int_0^{lo_i} p^(1/3), times (2n)^(1/3)
    uint32_t chunk_count[16];              // per 64 consecutive bins
    double chunk_h[16];
    double wave_tail[kParamsWaves];
    double tail_edge_log;                  // ln(1 + m/16) of the tail's first bin
    int tail_bin;
    float in13[SEARCH ? kNB : 1];          // BiScaled: (mass below bin i * lo_i^2)^(1/3), in fp32
};

template <int CTRL, int ROWS>
__device__ __forceinline__ float min_with_dpp(float v)
{
    return fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROWS, 0xf, false)));
}
__device__ __forceinline__ float wave_min(float v)
{
    v = min_with_dpp<0x111, 0xf>(v);
    v = min_with_dpp<0x112, 0xf>(v);
    v = min_with_dpp<0x114, 0xf>(v);
    v = min_with_dpp<0x118, 0xf>(v);
    v = min_with_dpp<0x142, 0xa>(v);
    v = min_with_dpp<0x143, 0xc>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Exclusive prefix sums over the bins: lane values v[k] of bins kParamsBlock k + tid.  On return v[k] is
// the sum over all bins below; the grand total is returned.  `chunk` is 16 entries of LDS that
// nobody else uses; one barrier.  `live`, bit k: some lane's v[k] is not 0.
template <typename T>
__device__ __forceinline__ T bin_scan(T (&v)[kBinsPerLane], uint32_t live, T* chunk)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    T incl[kBinsPerLane];
#pragma unroll
    for (int k = 0; k < kBinsPerLane; ++k) {
        incl[k] = v[k];
        if (live >> k & 1u) incl[k] = wave_scan(v[k]);
        if (lane == 63) chunk[kParamsWaves * k + wave] = incl[k];
    }
    __syncthreads();
    const T upto = row_scan(chunk[lane & 15]);
#pragma unroll
    for (int k = 0; k < kBinsPerLane; ++k) {
        const int c = kParamsWaves * k + wave;
        const T below = c > 0 ? lane_value(upto, c > 0 ? c - 1 : 0) : T(0);
        v[k] = below + (incl[k] - v[k]);
    }
    return lane_value(upto, 15);
}

// The density's integrals up to x, in fp64.
template <typename Lds>
struct DensityView {
    const Lds& L;
    double inv_n, absmax;
    // part of bin j below x, as a fraction of the bin; rw = 1 / its width
    __device__ __forceinline__ void covered(int j, double x, double& frac, double& rw) const
    {
        const double lo = bin_lo(j);
        double w;
        if (j < kNB - 1) {
            const int e = j > 0 ? ((j - 1) >> 4) - 44 : -40;
            w = ldexp(1.0, e);
            rw = ldexp(1.0, -e);
        } else {
            w = last_bin_width(absmax);
            rw = 1.0 / w;
        }
        double c = x - lo;
        c = c < 0.0 ? 0.0 : (c > w ? w : c);
        frac = c * rw;
    }
    // Q_U(a) and, in `elasticity`, dlnQ/dlna
    __device__ __forceinline__ double Q_U(double a, double& elasticity) const
    {
        const int j = bin_of(a);
        double frac, rw;
        covered(j, a, frac, rw);
        const auto bin = L.bins.at(j);
        const double h = (double)bin.here, mass = (double)bin.below + h * frac;
        elasticity = h * rw * a * recip(mass);
        return mass * inv_n;
    }
    // int_0^x p^(1/3) and, in `density`, p^(1/3) at x, both times (2n)^(1/3)
    __device__ __forceinline__ double half_int(double x, double& density) const
    {
        const int j = bin_of(x);
        double frac, rw;
        covered(j, x, frac, rw);
        const double below = L.H[j], mine = L.H[j + 1] - below;
        density = mine * rw;
        return below + mine * frac;
    }
    // Q_N(a) = (2 int_0^a p^(1/3))^3 / (4 a^2)
    __device__ __forceinline__ double Q_N(double a, double& elasticity) const
    {
        double density;
        const double half = half_int(a, density);
        elasticity = 3.0 * a * density * recip(half) - 2.0;
        const double u = half * recip(a);
        return u * u * half * inv_n;
    }
    // The same for a in bins 1 .. 896, to the same bits: the bin, the fraction of it below a and a / (its width) = 16 + m + fraction
    // are fields of a.  It shortens the chain of a step of the plain iteration, of which a record that contracts slowly takes 100
    // (1 such record 49.3 -> 41.5 us a launch, 952 records with some 51.3 -> 43.5).  The same detour avoided in the fp32 steps: 40.6 and
    // 42.5, but 2736 records without 21.3 -> 21.7, 391 13.4 -> 13.7: not done.
    __device__ __forceinline__ double Q_N_inner(double a, double& elasticity) const
    {
        uint32_t hi = (uint32_t)__double2hiint(a), lo = (uint32_t)__double2loint(a);
        asm("" : "+v"(hi), "+v"(lo));                          // kept out of the scalar unit, whose detour is longer
        const double* at = &L.H[(hi >> 16) - (((1023 - 40) << 4) - 1)];
        const double below = at[0], upto = at[1];
        const double frac = __hiloint2double((int)((__builtin_amdgcn_alignbit(hi, lo, 28) & 0xFFFFFu) | 0x3FF00000u), (int)(lo << 4)) - 1.0;
        const double mant = __hiloint2double((int)((hi & 0xFFFFFu) | 0x40300000u), (int)lo), r = recip(a);
        const double mine = upto - below, half = below + mine * frac, u = half * r;
        elasticity = 3.0 * mant * mine * recip(half) - 2.0;
        return u * u * half * inv_n;
    }
    __device__ __forceinline__ double inv_half_int(double t) const     // smallest x with int_0^x p^(1/3) >= t
    {
        // i with H[i] < t <= H[i+1], the smallest of those that are met: three rounds of independent reads, 64, 8 and 1 bins
        // apart, instead of ten of one read each (1 record 7.0 -> 6.8 us, 400 8.1 -> 7.9).  Each round goes on below the
        // first of its reads that is not below t, which keeps H[lo] < t <= the next one also where H is not monotone: its
        // sums are added in an order that depends on the lane, and over empty bins they differ by an ulp.
        int lo = 0, n = 14;
#pragma unroll
        for (int m = 14; m >= 1; --m) n = L.H[64 * m] < t ? n : m - 1;
        lo = 64 * n;
#pragma unroll
        for (int step = 8; step >= 1; step >>= 3) {
            n = 7;
#pragma unroll
            for (int m = 7; m >= 1; --m) n = L.H[lo + step * m < kNB ? lo + step * m : kNB] < t ? n : m - 1;
            lo += step * n;
        }
        if (lo >= kNB) return 65536.0 + last_bin_width(absmax);
        const double w = lo < kNB - 1 ? ldexp(1.0, lo > 0 ? ((lo - 1) >> 4) - 44 : -40) : last_bin_width(absmax);
        return bin_lo(lo) + w * ((t - L.H[lo]) / (L.H[lo + 1] - L.H[lo]));     // H[lo] < t <= H[lo + 1]
    }
};

// The fixed-point iteration a -> F(a) of the boxed equations converges near its fixed point like
// r^k, r being the logarithmic slope of F there.  Wherever it is sure to meet kRelTol within
// kMaxIter steps its limit is the fixed point, however that is computed: the slope at two points in
// a row and at the end is at most kCertifiedSlope, the steps have come down to kNearStep octaves
// after `plain` steps of the iteration itself, and the steps that are left, log(kNearStep / kRelTol) /
// log(1 / r), bring the sum to no more than kSureSteps.
constexpr float kCertifiedSlope = 0.75f;
constexpr float kNearStep = 0.02f;
constexpr int kSeekSteps = 60;
constexpr float kSureSteps = 90.0f;
__device__ __forceinline__ bool certified_slope(float r) { return fabsf(r) <= kCertifiedSlope; }

// One record.  WIDE: its counts may add up to more than 32 bits hold.
template <int GRID, bool WIDE>
__device__ __forceinline__ void design(ParamsLds<GRID != TQ_GRID_UNIFORM, WIDE, GRID == TQ_GRID_BISCALED>& L, const tq_stats_t* __restrict__ S, int bits,
                                       float alpha_override, tq_params_t* __restrict__ P)
{
    constexpr bool kRoots = GRID != TQ_GRID_UNIFORM;       // the integral of p^(1/3) is needed
    constexpr bool kBiscaled = GRID == TQ_GRID_BISCALED;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    uint32_t h[kBinsPerLane], cum[kBinsPerLane];           // of the lane's bins, unless WIDE
    if constexpr (!WIDE) {
#pragma unroll
        for (int k = 0; k < kBinsPerLane; ++k) {
            const int i = kParamsBlock * k + tid;
            h[k] = i < kNB ? S->hist[i] : 0u;
        }
    }
    // bit k: some of the wavefront's bins k count something.  A record of 16,384 elements leaves most of the 15 groups of 64 bins
    // empty, and thousands of records are bound by how many instructions they issue: empty groups are left out of the scans, the
    // search for the tail's bin and its logarithms (2736 records uniform 10.1 -> 9.4 us, non-uniform 22.7 -> 21.5, BiScaled of 768
    // 15.9 -> 15.4; 4 records non-uniform 7.4 -> 7.3)
    uint32_t live = (1u << kBinsPerLane) - 1u;
    const double centre_log = kOctaveLogs.centre[(tid - 1) & 15], edge_log = kOctaveLogs.edge[(tid - 1) & 15];
    const double absmax = (double)S->absmax;
    const float given_g_min = S->g_min;
    const uint64_t given_n_tail = S->n_tail;
    const double given_sum_log = S->sum_log_tail;
    const bool fixed_gmin = given_g_min > 0.0f;
    if (tid == 0) L.tail_bin = kNB;

    // Counts below each bin.  Without a caller-fixed g_min the tail starts at the lower edge of the first bin at
    // which the cumulative count reaches the 0.9-quantile of |g|: exactly one bin has the
    // count below the mark before it and at or above the mark with it.
    double n;
    if constexpr (WIDE) {
        if (wave == 0) {                                   // one wavefront, 64 bins at a time
            double sum = 0.0;
#pragma unroll 1
            for (int i = lane; i < 64 * ((kNB + 63) / 64); i += 64) {
                const double here = i < kNB ? (double)S->hist[i] : 0.0, upto = wave_scan(here);
                if (i < kNB) L.bins.cum[i] = sum + (upto - here);
                sum += lane_value(upto, 63);
            }
            if (lane == 0) L.bins.cum[kNB] = sum;
        }
        __syncthreads();
        n = L.bins.cum[kNB];
#pragma unroll 1
        for (int i = tid; i < kNB; i += kParamsBlock) {
            if (10.0 * L.bins.cum[i] < 9.0 * n && 10.0 * L.bins.cum[i + 1] >= 9.0 * n) {
                L.tail_bin = i;
                L.tail_edge_log = i < kNB - 1 ? edge_log : 0.0;
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < kBinsPerLane; ++k) {
            cum[k] = h[k];
            if (__builtin_amdgcn_ballot_w64(h[k] != 0u) == 0ull) live &= ~(1u << k);
        }
        const uint32_t n_count = bin_scan(cum, live, L.chunk_count);
        n = (double)n_count;
#pragma unroll
        for (int k = 0; k < kBinsPerLane; ++k) {
            const int i = kParamsBlock * k + tid;
            if (i < kNB) L.bins.hc[i] = make_uint2(h[k], cum[k]);
            if (!(live >> k & 1u)) continue;
            const uint64_t mark = 9ull * n_count;
            if (10ull * cum[k] < mark && 10ull * ((uint64_t)cum[k] + h[k]) >= mark) {
                L.tail_bin = i;
                L.tail_edge_log = i < kNB - 1 ? edge_log : 0.0;
            }
        }
    }
    __syncthreads();
    int tail_bin = L.tail_bin;
    double g_min;
    if (fixed_gmin) { g_min = (double)given_g_min; tail_bin = kNB; }
    else if (tail_bin >= kNB) { g_min = 0.0; }
    else g_min = bin_lo(tail_bin);                         // 0 when the quantile sits in bin 0
    const bool binned_tail = !fixed_gmin && g_min > 0.0;
    const double inv_n = n > 0.0 ? recip(n) : 0.0;

    // density^(1/3) (times (2n)^(1/3), which cancels or is put back where it is used), its integral up
    // to each bin, and the binned log-sum of the tail
    double sum_log_binned = 0.0;
    if (binned_tail) {
        const int octave0 = (tail_bin - 1) >> 4;
        double local_t = 0.0;
#pragma unroll
        for (int k = 0; k < kBinsPerLane; ++k) {
            if (!(live >> k & 1u)) continue;
            const int i = kParamsBlock * k + tid;
            const double from_octave = i < kNB - 1 ? centre_log : 0.0;
            double here = 0.0;
            if constexpr (!WIDE) here = (double)h[k];
            else if (i < kNB) here = (double)S->hist[i];
            if (i >= tail_bin)
                local_t += here * ((double)(((i - 1) >> 4) - octave0) * kLn2 + (from_octave - L.tail_edge_log));
        }
        local_t = wave_scan(local_t);
        if (lane == 63) L.wave_tail[wave] = local_t;
    }
    if constexpr (kRoots) {
        double pw[kBinsPerLane];
        // one bin after the other (a loop, not unrolled: its code is fetched once), through LDS
#pragma unroll 1
        for (int i = tid; i < kNB; i += kParamsBlock) {
            const auto count = L.bins.at(i).here;
            double c = 0.0;
            if (__builtin_amdgcn_ballot_w64(count != 0) != 0ull) {
                // (count / w)^(1/3) w = count^(1/3) w^(2/3); the bin is w = 2^e wide, e = 3 third + rem
                c = cube_root((double)count);
                if (i < kNB - 1) {
                    const int e = i > 0 ? ((i - 1) >> 4) - 44 : -40;
                    const int third = (e + 63) / 3 - 21, rem = e - 3 * third;
                    c = ldexp(c * (rem == 0 ? 1.0 : (rem == 1 ? 1.58740105196819947475 : 2.51984209978974632953)), 2 * third);
                } else if (count != 0) {
                    const double wr = cube_root(last_bin_width(absmax));
                    c = c * wr * wr;
                }
            }
            L.H[i] = c;
            if constexpr (kBiscaled) {
                const float inside = (float)L.bins.at(i).below * (float)inv_n;
                L.in13[i] = inside > 0.0f ? exp2_hw((log2_hw(inside) + 2.0f * log2_hw((float)bin_lo(i))) * (1.0f / 3.0f)) : 0.0f;
            }
        }
#pragma unroll
        for (int k = 0; k < kBinsPerLane; ++k) pw[k] = kParamsBlock * k + tid < kNB ? L.H[kParamsBlock * k + tid] : 0.0;
        const double all = bin_scan(pw, live, L.chunk_h);
#pragma unroll
        for (int k = 0; k < kBinsPerLane; ++k) {
            const int i = kParamsBlock * k + tid;
            if (i < kNB) L.H[i] = pw[k];
        }
        if (tid == 0) L.H[kNB] = all;
    }
    __syncthreads();
    if (binned_tail) {
#pragma unroll
        for (int w = 0; w < kParamsWaves; ++w) sum_log_binned += L.wave_tail[w];
    }
    if (wave != 0) return;                                 // one wavefront goes on, every lane with the same scalars

    const DensityView<ParamsLds<kRoots, WIDE, kBiscaled>> D{L, inv_n, absmax};

    // BiScaled search: the edge lo_j < a (j = 0: beta = 0) that minimises Q_B(a, lo_j / a) =
    // v^3, v = ((mass outside beta) (1 - k)^2)^(1/3) + ((mass inside) k^2)^(1/3), the smallest such edge on a tie.
    // One wavefront, a lane per edge, windows of 64 edges (four octaves) from a's bin downwards.  The first summand grows
    // towards smaller edges: the search ends where it alone is above the best v, nearly always within the two windows
    // that are looked at at once.
    constexpr int kAtOnce = 2;
    struct Edge { float v, s1, mass, rest, lo, in; };
    struct Threshold { float a, inv_a16, inv_a23, part; int bin; decltype(L.bins.at(0).below) below; };
    auto edge_of = [&](int window, const Threshold& A) {
        const int i = A.bin - 64 * window - lane, j = i > 0 ? i : 0;
        Edge e;
        e.lo = i > 0 ? __uint_as_float((uint32_t)(i + 1391) << 19) : (i == 0 ? 0.0f : __builtin_inff());
        // mass between the edge and a, from an exact difference of counts; 1 - k of the formula
        e.mass = ((float)(A.below - L.bins.at(j).below) + A.part) * (float)inv_n;
        e.rest = (0.0625f * (A.a - e.lo)) * A.inv_a16;
        e.in = L.in13[kBiscaled ? j : 0] * A.inv_a23;
        e.s1 = exp2_hw(log2_hw(e.mass * (e.rest * e.rest)) * (1.0f / 3.0f));
        e.v = e.lo < A.a ? e.s1 + e.in : __builtin_inff();
        return e;
    };
    // the fp32 search at threshold a: min_k v, and the elasticity of Q_B = v^3 in a with the best edge held
    // fixed; v_f keeps the first candidates, `windows` is how many were looked at
    float v_f[kAtOnce];
    int windows = 0;
    Threshold at_a = {};
    auto search_f = [&](float a, float& elasticity, auto inner) {
        constexpr bool INNER = decltype(inner)::value;     // a is in bins 1 .. 896
        const uint32_t bits_a = __float_as_uint(a);
        int ja = (int)(bits_a >> 19) - 1391;
        ja = ja < 0 ? 0 : (ja > kNB - 1 ? kNB - 1 : ja);
        // fraction of a's bin below a, and d(fraction)/d(ln a) = a / (bin width)
        float frac, per_ln;
        if (INNER || (ja >= 1 && ja < kNB - 1)) {
            frac = (float)(bits_a & 0x7FFFFu) * (1.0f / 524288.0f);
            per_ln = __uint_as_float((bits_a & 0x7FFFFFu) | 0x41800000u);
        } else {
            double f, rw;
            D.covered(ja, (double)a, f, rw);
            frac = (float)f;
            per_ln = (float)(rw * (double)a);
        }
        const auto bin = L.bins.at(ja);
        // 16 / a: the hardware's reciprocal has no subnormal results, which 1 / a is from 2^126 on
        at_a = Threshold{a, rcp_hw(0.0625f * a), exp2_hw(log2_hw(a) * (-2.0f / 3.0f)), (float)bin.here * frac,
                         __builtin_amdgcn_readfirstlane(ja), bin.below};
        Edge best = edge_of(0, at_a), e = best;
        v_f[0] = best.v;
#pragma unroll
        for (int w = 1; w < kAtOnce; ++w) {
            e = edge_of(w, at_a);
            v_f[w] = e.v;
            if (e.v <= best.v) best = e;
        }
        float m = wave_min(best.v);
        windows = kAtOnce;
        while (at_a.bin >= 64 * windows && !(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(e.s1), 63)) > m * 1.0002f)) {
            e = edge_of(windows++, at_a);
            if (e.v <= best.v) best = e;
            m = wave_min(best.v);
        }
        // v = s1 + s2: d ln(s1) = dmass / (3 mass) + 2/3 k / (1 - k), d ln(s2) = -2/3
        const float d1 = best.mass > 0.0f ? (float)bin.here * per_ln * (float)inv_n * rcp_hw(best.mass) + 0.125f * best.lo * at_a.inv_a16 * rcp_hw(best.rest) : 0.0f;
        const float slope = (best.s1 * d1 - 2.0f * best.in) * rcp_hw(best.v);
        const unsigned long long at = __builtin_amdgcn_ballot_w64(best.v == m);
        elasticity = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(slope), at ? __builtin_ctzll(at) : 0));
        return m;
    };
    // the search in fp64, over the edges whose fp32 value is within 1e-4 of the fp32 minimum (its error is
    // below 1e-5: the masses are differences of exact counts, every other term is good to a few ulp).  Nearly always that
    // is one edge, and where only the edge is asked for the search ends with it.
    int best_bin = 0;
    bool only_one = false;                                 // no other is within 1e-5: it is the best edge at a rounded to fp32, too
    auto search_d = [&](double a, double& elasticity, bool edge_only = false) {
        float el;
        const float a_f = (float)a, bound = search_f(a_f, el, std::false_type{}) * 1.0001f;
        auto close_ones = [&](int window, float v32) {     // an edge between a and a rounded to fp32 counts as close
            const int i = at_a.bin - 64 * window - lane;
            const double lo = i >= 0 ? bin_lo(i) : __builtin_inf();
            return (unsigned long long)__builtin_amdgcn_ballot_w64(lo < a && (v32 <= bound || !(lo < (double)a_f)));
        };
        if (edge_only && windows == kAtOnce) {
            const unsigned long long c0 = close_ones(0, v_f[0]), c1 = close_ones(1, v_f[1]);
            only_one = __builtin_popcountll(c0) + __builtin_popcountll(c1) == 1;
            if (only_one) {
                best_bin = at_a.bin - (c0 ? __builtin_ctzll(c0) : 64 + __builtin_ctzll(c1));
                return 0.0;
            }
        }
        const int ja = bin_of(a);
        double frac, rw;
        D.covered(ja, a, frac, rw);
        const auto bin = L.bins.at(ja);
        const double part = (double)bin.here * frac, inv_a = recip(a);
        double q = 1.0e300, second = 1.0e300;
        int jbest = 0;
#pragma unroll 1
        for (int window = 0; window < windows; ++window) {
            float v32 = window == 0 ? v_f[0] : v_f[1];
            if (window >= kAtOnce) v32 = edge_of(window, at_a).v;
            unsigned long long left = close_ones(window, v32);
            if (left == 0ull) continue;
            const int i = at_a.bin - 64 * window - lane, j = i > 0 ? i : 0;
            const double lo = bin_lo(j);
            const auto below = L.bins.at(j).below;
            const double kk = lo * inv_a, rest = (a - lo) * inv_a;
            const double out_mass = ((double)(bin.below - below) + part) * inv_n, in_mass = (double)below * inv_n;
            const double v = cube_root(out_mass * rest * rest) + cube_root(in_mass * kk * kk);
            while (left) {                                 // a few candidates, in descending order
                const int l = __builtin_ctzll(left);
                left &= left - 1;
                const double vl = lane_value(v, l);
                second = vl <= q ? q : (vl < second ? vl : second);
                if (vl <= q) { q = vl; jbest = at_a.bin - 64 * window - l; }
            }
        }
        best_bin = jbest;
        only_one = second > q * 1.00001;
        // the elasticity of the edge that won here: near a tie the fp32 search may have taken another one's
        const double lo = bin_lo(jbest), rest = (a - lo) * inv_a;
        const double below = (double)L.bins.at(jbest).below, mass = ((double)bin.below - below + part) * inv_n;
        const float inside = (float)(below * inv_n), kk = (float)(lo * inv_a);
        const float s2 = inside > 0.0f ? exp2_hw((log2_hw(inside) + 2.0f * log2_hw(kk)) * (1.0f / 3.0f)) : 0.0f;
        const float d1 = mass > 0.0 ? (float)((double)bin.here * rw * a * inv_n) * rcp_hw((float)mass) + 2.0f * kk * rcp_hw((float)rest) : 0.0f;
        elasticity = (double)((((float)q - s2) * d1 - 2.0f * s2) * rcp_hw((float)q));
        return q * q * q;
    };
    bool inner = false;                                    // every a is in bins 1 .. 896
    // Q of the family at a, and dlnQ/dlna
    auto Q = [&](double a, double& elasticity) {
        if constexpr (GRID == TQ_GRID_UNIFORM) return D.Q_U(a, elasticity);
        else if constexpr (kBiscaled) return search_d(a, elasticity);
        else return inner ? D.Q_N_inner(a, elasticity) : D.Q_N(a, elasticity);
    };
    // the same in fp32 for bins 1 .. 896: the fraction of the bin below a is a's low mantissa bits
    auto log2_Q_f = [&](float a, float& elasticity) {
        const uint32_t bits_a = __float_as_uint(a);
        int j = (int)(bits_a >> 19) - 1391;
        j = j < 1 ? 1 : (j > kNB - 2 ? kNB - 2 : j);
        const float frac = (float)(bits_a & 0x7FFFFu) * (1.0f / 524288.0f);
        const float mant = __uint_as_float((bits_a & 0x7FFFFFu) | 0x41800000u);    // a / (bin width) = 16 + m + frac
        if constexpr (GRID == TQ_GRID_UNIFORM) {
            const auto bin = L.bins.at(j);
            const float mass = (float)bin.below + (float)bin.here * frac;
            elasticity = (float)bin.here * mant * rcp_hw(mass);
            return log2_hw(mass * (float)inv_n);
        } else if constexpr (kBiscaled) {
            return 3.0f * log2_hw(search_f(a, elasticity, std::true_type{}));
        } else {
            const double below = L.H[j];
            const float mine = (float)(L.H[j + 1] - below), half = (float)below + mine * frac;
            elasticity = 3.0f * mine * mant * rcp_hw(half) - 2.0f;
            const float u = half * rcp_hw(a);
            return log2_hw(u * u * (half * (float)inv_n));
        }
    };

    const int s = (1 << bits) - 1;
    bool have_split = false;                               // BiScaled: best_bin belongs to alpha rounded to fp32
    uint32_t flags = 0;
    double gamma = 0.0, rho = 0.0, alpha;
    if (n <= 0.0 || absmax <= 0.0) {
        // nothing finite and non-zero to design from; a threshold the caller gives is still honoured
        flags |= TQ_F_DEGENERATE;
        alpha = kAlphaFloor;
        if (alpha_override > 0.0f) { flags |= TQ_F_ALPHA_OVERRIDE; alpha = (double)alpha_override; }
        g_min = 0.0;
    } else {
        double n_tail, sum_log;
        if (fixed_gmin) {
            n_tail = (double)given_n_tail;
            sum_log = given_sum_log;
        } else {
            n_tail = g_min > 0.0 ? n - (double)L.bins.at(tail_bin).below : 0.0;
            sum_log = g_min > 0.0 ? sum_log_binned : 0.0;
        }
        const bool tail_ok = g_min > 0.0 && n_tail > 0.0 && sum_log > 0.0 && g_min < absmax;
        if (tail_ok) {
            gamma = 1.0 + n_tail * recip(sum_log);
            rho = n_tail * 0.5 * inv_n;
        }
        if (alpha_override != 0.0f) {
            flags |= TQ_F_ALPHA_OVERRIDE;
            alpha = alpha_override > 0.0f ? (double)alpha_override : absmax;
        } else if (!tail_ok) {
            flags |= TQ_F_DEGENERATE;
            alpha = absmax;
        } else {
            double gu = gamma;
            if (gu < kGammaFloor) { gu = kGammaFloor; flags |= TQ_F_GAMMA_CLAMPED; }
            const double a_min = g_min * (1.0 + 0.0009765625), a_max = absmax;
            inner = a_min >= kFirstEdge && a_max < 65536.0;
            const double C = 2.0 * rho * (double)(s * s) * recip(gu - 2.0);
            const double ex = recip(gu - 1.0);
            auto clampa = [&](double a) { a = a > a_min ? a : a_min; return a < a_max ? a : a_max; };
            double a = 0.0;
            bool converged = false;

            // fp32: t = log2(a / g_min), t -> f(t) = ex (log2 C - log2 Q).  Plain steps, as the definition
            // takes them, until two slopes in a row are certified and the step is below a third of a bin; then
            // Newton steps.  (The last bin, 65536 and up, spans octaves and is left to the plain path.)
            if (a_max < 65536.0) {
                const float exf = (float)ex, log2_C = log2_hw((float)C), g_f = (float)g_min;
                const float t_min = log2_hw((float)(1.0 + 0.0009765625)), t_max = log2_hw((float)(a_max / g_min));
                auto clampt = [&](float t) { t = t > t_min ? t : t_min; return t < t_max ? t : t_max; };
                float t = clampt(exf * log2_C), r_before = 2.0f, plain = 0.0f;
                bool near = false;
                for (int it = 0; it < kSeekSteps && !near; ++it) {
                    float el;
                    const float f = exf * (log2_C - log2_Q_f(g_f * exp2_hw(t), el));
                    const float r = -exf * el;
                    float step = clampt(f) - t;
                    if (certified_slope(r) && certified_slope(r_before) && fabsf(step) <= kNearStep)
                        step = clampt(t + (f - t) * rcp_hw(1.0f - r)) - t;
                    else
                        plain = (float)it;
                    r_before = r;
                    t += step;
                    near = fabsf(step) <= 1e-5f;
                }
                // fp64: Newton on ln(a / g_min) + ex ln(Q / C); two steps end it nearly always
                a = t >= t_max ? a_max : clampa(g_min * (double)exp2_hw(t));
                for (int it = 0; it < 5 && near && !converged; ++it) {
                    double el;
                    have_split = false;
                    const double q = Q(a, el);
                    if (!(q > 0.0)) break;
                    const double part = ln(((lane & 1) ? q : a) * recip((lane & 1) ? C : g_min));    // the two logarithms at once, in even and odd lanes
                    const double residual = lane_value(part, 0) + ex * lane_value(part, 1), slope = -ex * el;
                    const double delta = -residual * (double)rcp_hw((float)(1.0 - slope));
                    const double an = clampa(a * (1.0 + delta * (1.0 + 0.5 * delta)));
                    if ((a >= a_max && residual <= 0.0) || (a <= a_min && residual >= 0.0)) { converged = true; break; }
                    const float r = fabsf((float)slope);
                    if (!certified_slope(r) || !(fabs(delta) < 0.03)) break;
                    if (plain + 27.6f * rcp_hw(-log2_hw(r)) > kSureSteps) break;   // log2(kNearStep / kRelTol) = 27.6
                    // quadratic convergence inside a bin: what is left is of the order of delta^2
                    converged = fabs(delta) <= 1e-5 && bin_of(an) == bin_of(a);
                    if constexpr (kBiscaled) {
                        // and where the best edge changes Q_B has a kink: it has to be the same at the end of the step
                        const int from = best_bin;
                        if (converged) (void)search_d(an, el, true);
                        have_split = converged && only_one;
                        converged = (converged && best_bin == from) || fabs(residual) <= kRelTol;
                    }
                    a = an;
                }
            }
            if (!converged) {
                // the definition's iteration, step by step
                have_split = false;
                const double log_c = ln(C);
                auto power = [](double x) { return WIDE ? exp_by_ln(x) : exp(x); };
                a = clampa(g_min * power(ex * log_c));     // alpha' of Sec. IV-A (Q = 1)
                for (int it = 0; it < kMaxIter; ++it) {
                    double el;
                    const double q = Q(a, el);
                    // (C/q)^ex evaluated as exp(ex (ln C - ln q))
                    const double next = fmin(fmax(g_min * power(ex * (log_c - ln(q))), a_min), a_max), an = q > 0.0 ? next : a_max;
                    const bool done = __builtin_amdgcn_ballot_w64(fabs(an - a) <= kRelTol * an) != 0ull;   // the same in every lane
                    a = an;
                    if (done) { converged = true; break; }
                }
            }
            if (!converged) flags |= TQ_F_NOT_CONVERGED;
            if (a >= a_max) flags |= TQ_F_ALPHA_CLAMPED_MAX;
            else if (a <= a_min) flags |= TQ_F_ALPHA_CLAMPED_MIN;
            alpha = a;
        }
    }

    // the codebook, a lane per level
    const float alpha_f = (float)(alpha > kAlphaFloor ? alpha : kAlphaFloor);
    const double af = (double)alpha_f;
    double half = 0.0;
    if constexpr (kRoots) {
        double density;
        half = D.half_int(af, density);
    }
    if constexpr (kBiscaled) {
        double el;
        if (half > 0.0 && !have_split) (void)search_d(af, el, true);   // the split belongs to the rounded threshold
    }
    const int k = lane;                                    // this lane's level, 0 .. s
    float lv = 0.0f;
    if (GRID == TQ_GRID_UNIFORM || !(half > 0.0) || (kBiscaled && best_bin == 0)) {
        lv = (float)(-af + (double)k * (2.0 * af / (double)s));
    } else if constexpr (kBiscaled) {
        const double beta = bin_lo(best_bin), kk = beta / af;
        double el;
        const double c_b = (double)L.bins.at(best_bin).below * inv_n, c_a = D.Q_U(af, el);
        const double p1 = c_b / (2.0 * beta);
        const double rest = c_a - c_b > 0.0 ? c_a - c_b : 0.0;
        const double p2 = rest / (2.0 * (af - beta));
        const double inner = cbrt(p1) * kk, outer = cbrt(p2) * (1.0 - kk);
        const double x = inner + outer > 0.0 ? (double)s * inner / (inner + outer) : (double)s;
        int s_beta = 2 * (int)floor((x - 1.0) * 0.5 + 0.5) + 1;           // nearest odd integer
        s_beta = s_beta < 1 ? 1 : (s_beta > s - 2 ? s - 2 : s_beta);
        const int out_cells = (s - s_beta) / 2;                            // cells beyond beta on each side
        const int j = k - out_cells;
        if (j > 0 && j < s_beta) {
            lv = (float)(-beta + (double)j * (2.0 * beta / (double)s_beta));
        } else {
            const int beyond = j <= 0 ? -j : j - s_beta;                   // cells from beta outwards
            const float xo = (float)(beta + (double)beyond * ((af - beta) / (double)out_cells));
            lv = j <= 0 ? -xo : xo;
        }
    } else if constexpr (kRoots) {
        const int up = k > s / 2 ? k : s - k;                              // the positive one of a mirrored pair
        double x = D.inv_half_int(half * (double)(2 * up - s) / (double)s);
        x = x < af ? x : af;
        lv = k > s / 2 ? (float)x : -(float)x;
    }
    if (k == 0) lv = -alpha_f;
    if (k == s) lv = alpha_f;
    if (k > s) lv = 0.0f;
    const float next = __shfl_down(lv, 1, 64);
    float iw = 0.0f;
    if (k < s) {
        if (GRID == TQ_GRID_UNIFORM) {
            iw = (float)((double)s / (2.0 * af));
        } else {
            const double width = (double)next - (double)lv;
            if (width > 0.0) {
                const double r = 1.0 / width;
                iw = r <= 3.4028234663852886e38 ? (float)r : 0.0f;
            }
        }
    }
    if (lane < 16) {
        P->level[lane] = lv;
        P->inv_w[lane] = iw;
    }
    if (lane == 0) {
        P->alpha = alpha_f;
        P->bits = (uint32_t)bits;
        P->s = (uint32_t)s;
        P->grid = (uint32_t)GRID;
        P->gamma_hat = (float)gamma;
        P->rho_hat = (float)rho;
        P->g_min = (float)g_min;
        P->flags = flags;
    }
}

template <int GRID>
__global__ __launch_bounds__(kParamsBlock) void tq_params_kernel(const PtrTable stats_tab, uint32_t nb, int bits,
                                                           float alpha_override, const MutPtrTable params_tab)
{
    constexpr bool kRoots = GRID != TQ_GRID_UNIFORM;
    __shared__ union Lds {
        ParamsLds<kRoots, false, GRID == TQ_GRID_BISCALED> narrow;
        ParamsLds<kRoots, true, GRID == TQ_GRID_BISCALED> wide;
        __device__ Lds() {}
    } L;
    // one workgroup per bucket, blockIdx.y = tensor of the batch
    const uint32_t bucket = linear_block();
    if (bucket >= nb) return;
    const tq_stats_t* __restrict__ S = static_cast<const tq_stats_t*>(stats_tab.p[blockIdx.y]) + bucket;
    tq_params_t* __restrict__ P = static_cast<tq_params_t*>(params_tab.p[blockIdx.y]) + bucket;
    if (__builtin_expect((S->n >> 32) == 0, 1)) design<GRID, false>(L.narrow, S, bits, alpha_override, P);
    else design<GRID, true>(L.wide, S, bits, alpha_override, P);
}

}  // namespace tq

// Host side of tq_params / tq_params_multi after the argument checks of the C entry points.
hipError_t tq_launch_params(const tq_stats_t* const* stats, int count, uint64_t nb, int bits, int grid,
                            float alpha_override, tq_params_t* const* params, hipStream_t st)
{
    dim3 blocks;
    if (count < 1 || count > tq::kMaxBatch || !tq::fold_grid(nb, tq::kParamsBlock, (unsigned)count, blocks))
        return hipErrorInvalidValue;
    tq::PtrTable stt{};
    tq::MutPtrTable pt{};
    for (int i = 0; i < count; ++i) { stt.p[i] = stats[i]; pt.p[i] = params[i]; }
#define TQ_LAUNCH_PARAMS(G) \
    hipLaunchKernelGGL(tq::tq_params_kernel<G>, blocks, dim3(tq::kParamsBlock), 0, st, stt, (uint32_t)nb, bits, alpha_override, pt)
    switch (grid) {
        case TQ_GRID_UNIFORM: TQ_LAUNCH_PARAMS(TQ_GRID_UNIFORM); break;
        case TQ_GRID_NONUNIFORM: TQ_LAUNCH_PARAMS(TQ_GRID_NONUNIFORM); break;
        default: TQ_LAUNCH_PARAMS(TQ_GRID_BISCALED); break;
    }
#undef TQ_LAUNCH_PARAMS
    return hipGetLastError();
}
