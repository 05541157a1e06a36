// Fused vocabulary-wide softmax + lossless rejection sampling (the rejection procedure the
// paper's Section 2.1 relies on; acceptance length as defined in its Section 2.2).
//
// Two launches per step, the vocabulary cut into SAMP_PARTS ranges so that a batch of a few dozen
// sequences still occupies the whole chip (one workgroup per row or sequence left 7/8 of the CUs idle):
//   1. row_stats_kernel: workgroup = (logits row, range) -> (reference, sum of exp) of logits / T over the range;
//   2. reject_scan_kernel: workgroup = (sequence, range): the accept tests side by side (every range's workgroup
//      repeats them and arrives at the same n), then the exponential race over its range of the single row that
//      decides the emitted token (residual row at the first rejection, bonus row after k acceptances) -> the range's
//      best key; the workgroup that finishes a sequence last takes the best key over the ranges, ties to the lowest
//      token -> outputs.
// Only the rows' statistics, the k probed q entries and one q row are read: (k+1+2) V floats
// per sequence at most.
#include <mutex>

#include "common.h"

namespace specv {

constexpr int SAMP_THREADS = 512;
constexpr int SAMP_WAVES = SAMP_THREADS / 64;
constexpr int SAMP_GPT = 4;                   // groups of 4 entries a thread holds in registers at a time

struct Philox4 { uint32_t x, y, z, w; };

__device__ inline Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;   // one multiply each for both halves
        c0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
        c1 = (uint32_t)p1;
        c2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return Philox4{c0, c1, c2, c3};
}

constexpr int SAMP_PARTS = 8;                 // ranges the vocabulary is cut into (whole groups of 4 entries: one Philox call each)

// groups of 4 vocabulary entries of range `part`: [g0, g1)
__device__ inline void part_groups(int V, int part, int* g0, int* g1)
{
    const int groups = (V + 3) >> 2, per = (groups + SAMP_PARTS - 1) / SAMP_PARTS;
    *g0 = part * per < groups ? part * per : groups;
    *g1 = (part + 1) * per < groups ? (part + 1) * per : groups;
}

// Everything a decision hangs on is fp64, as the definition has it: z = logit / T, e = exp(z - max), p = e / sum, the accept
// test u * q < p, the race keys w / (-ln u).  In the accept tests and the keys z is a division; in the sums and in the q that is
// written out z - max is (logit - largest) * (1 / T), whose first factor is exact and whose error, 2^-52 of itself, is that of the
// two divisions.  With fp32 keys two candidates closer than 1e-6 relative could swap, and a residual p - q that cancels to a few
// ulps was noise; in fp64 the choice differs from an fp64 reference's only where its own keys agree to 15 digits.
//
// What keeps that cheap (both kernels should be bound by reading the logits):
//   * the sums need an fp64 exponential per entry: exp_sum below, 15 fp64 instructions, no branch, no special cases;
//   * a race needs its keys in fp64 only where they can win: every entry's key is first bounded in fp32 from above and
//     below, and the entries whose upper bound reaches the best lower bound known to the wavefront are then evaluated in fp64.
//     Those are few unless the weights cancel: a residual that is rounding noise everywhere (q = p) leaves every entry.
// Measured (V = 128256): figures at the kernels.

// a * b + c with c in scalar registers.  Left to itself the compiler takes the two-address form and copies the constant into
// the result first, which doubles the instructions of a polynomial.
__device__ inline double fma_const(double a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// exp(x) for x <= 0, without a branch: x = n ln 2 + r, |r| <= ln 2 / 2, 1 + r + r^2 / 2 + r^3 p(r) with p of degree 8 interpolating
// (e^r - 1 - r - r^2 / 2) / r^3 at the Chebyshev nodes of that range (error 3.4e-17 of e^r; Taylor to r^12, one term more, 2.3e-16), 2^n through the
// exponent bits.  The rounding of ln 2 to a double adds n 2.3e-17: an ulp at n = 10, and a term of a sum that small weighs 2^-n.
// Arguments below -708 (and NaN) count as -708: 3e-308, nothing beside the largest term of 1.
__device__ inline double exp_sum(double x)
{
    const double magic = 6755399441055744.0;                         // 1.5 * 2^52: the sum's low bits are rint(x / ln 2)
    asm("v_max_f64 %0, %1, %2" : "=v"(x) : "v"(x), "s"(-708.0));
    const double t = __builtin_fma(x, 1.4426950408889634074, magic);
    const double n = t - magic;
    const double r = __builtin_fma(n, -0.6931471805599453094, x);
    double p = fma_const(r, 0x1.af2360e209be0p-26, 0x1.28803926c8ebbp-22);
    p = fma_const(p, r, 0x1.71de17e7960e6p-19);
    p = fma_const(p, r, 0x1.a019c9ab213aap-16);
    p = fma_const(p, r, 0x1.a01a01a4b26e2p-13);
    p = fma_const(p, r, 0x1.6c16c1738ecf7p-10);
    p = fma_const(p, r, 0x1.1111111110e6bp-7);
    p = fma_const(p, r, 0x1.5555555554cb8p-5);
    p = fma_const(p, r, 0x1.5555555555555p-3);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return __hiloint2double(__double2hiint(p) + (__double2loint(t) << 20), __double2loint(p));
}

// largest of the wavefront's values, in every lane: vector instructions only (a shuffle would take six trips through the LDS crossbar)
__device__ inline float wave_max(float x)
{
    unsigned u = __float_as_uint(x);
    auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    u = __float_as_uint(x);
    auto b = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    x = fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, false)));      // row_ror:8, 4, 2, 1
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xf, 0xf, false)));
    return fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xf, 0xf, false)));
}

// GPT groups of a lane: group u starts at entry 4 (gb + u * SAMP_THREADS + lane).  VEC: the row is 16-byte aligned and V a multiple of 4.  The loads go out
// together, with no branch between them: beyond group g1 the last group is read again, beyond entry V the last entry.
template <bool VEC, int GPT>
__device__ inline void load_round(const float* __restrict__ row, int gb, int g1, int V, float (&v)[GPT][4])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
        const int g = gb + u * SAMP_THREADS + lane, gc = g < g1 ? g : g1 - 1;
        if constexpr (VEC) {
            const float4 a = *(const float4*)(row + 4 * (int64_t)gc);
            v[u][0] = a.x; v[u][1] = a.y; v[u][2] = a.z; v[u][3] = a.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int at = 4 * gc + j;
                v[u][j] = row[at < V ? at : V - 1];
            }
        }
    }
}
// the same with `pad` in the place of what lies beyond
template <bool VEC>
__device__ inline void load_round(const float* __restrict__ row, int gb, int g1, int V, float pad, float (&v)[SAMP_GPT][4])
{
    load_round<VEC, SAMP_GPT>(row, gb, g1, V, v);
#pragma unroll
    for (int u = 0; u < SAMP_GPT; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int g = gb + u * SAMP_THREADS + (threadIdx.x & 63);
            if (!(g < g1 && (VEC || 4 * g + j < V))) v[u][j] = pad;
        }
}
// whether every row of an array can be read in 16-byte words
static bool rows_vec(const void* rows, int64_t stride, int V) { return ((uintptr_t)rows & 15) == 0 && (stride & 3) == 0 && (V & 3) == 0; }

// a value that every lane holds alike, in scalar registers: the scans have none of the vector ones to spare
__device__ inline double uniform(double x)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)), __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// groups per lane that the round starting at group gb holds (the same for a wavefront)
template <int GPT>
__device__ inline int round_groups(int gb, int g1)
{
    const int n = (g1 - gb + SAMP_THREADS - 1) / SAMP_THREADS;
    return n < GPT ? n : GPT;
}

// N lanes side by side (a power of two; every N-th lane's group of a wavefront for itself) hold (M_i, S_i); all get M = max M_i and
// S = sum_i S_i exp((M_i - M) / T), summed in a fixed order.
template <int N>
__device__ inline double2 merge_stats(double2 c, double rT)
{
    double M = c.x;
    for (int off = N / 2; off > 0; off >>= 1) M = fmax(M, __shfl_xor(M, off));
    double S = c.y > 0.0 ? c.y * exp_sum((c.x - M) * rT) : 0.0;
    for (int off = N / 2; off > 0; off >>= 1) S += __shfl_xor(S, off);
    return make_double2(M, S);
}

// a row's statistics from those of its ranges, SAMP_PARTS lanes a row (each with its range's): M = max m_p, S = sum_p s_p exp((m_p - M) / T).  M stays
// a logit: M / T is formed where it is needed, as M cannot be had back from it when T is infinite (0) or subnormal.  S = 0 says that the row has no
// distribution: it is -inf throughout, or holds +inf (exp_sum gives such a row's terms the value of exp(-708), not NaN).  Its
// probabilities are then NaN as 0 / 0 is: no accept test passes and no key is kept.
__device__ inline double2 row_stat(const double2* __restrict__ stats, int64_t row, double rT)
{
    const double2 st = merge_stats<SAMP_PARTS>(stats[row * SAMP_PARTS + (threadIdx.x & (SAMP_PARTS - 1))], rT);
    return make_double2(st.x, st.x == INFINITY ? 0.0 : st.y);
}

// (largest logit, sum of exp((logit - largest) / T)) of one range of a row.  Each wavefront reads its entries once, STAT_GPT groups of 4 per lane
// at a time (for vocabularies of up to 131072 all of them), takes the maximum of what is in registers as the reference (moving it, and what has been
// summed, when a later round exceeds it), so there is no second pass over the logits and no barrier before the sums; the wavefronts' pairs are
// merged in a fixed order.
// Bound by its vector instructions (21 per entry, 19 of them fp64 at the fp32 rate: 15 of the exponential, the conversion, difference, scaling and sum) with the reads beside them; 384 rows of 128256 take 47 us = 4.2 TB/s, 1024 rows
// 118 (55 and 140 on the same boxes with a Taylor series of one term more, two rounds a wavefront and a serial merge; 122 and 355 as two passes with the library's exponential).
// (zero_rows != null: the workgroup also clears its eighth of row blockIdx.x of that array, zero_width entries wide - the
// q rows a mapped draft draw then fills at scattered positions; counters != null: the sequences' arrival counters of the
// scan that follows, counter_rows rows per sequence)
constexpr int STAT_GPT = 8;
template <bool VEC>
__global__ __launch_bounds__(SAMP_THREADS) void row_stats_kernel(const float* __restrict__ logits, int64_t row_stride, int V, double rT,
                                                                  double2* __restrict__ stats, int32_t* __restrict__ counters,
                                                                  int counter_rows, float* __restrict__ zero_rows = nullptr,
                                                                  int64_t zero_stride = 0, int zero_width = 0)
{
    if (blockIdx.y == 0 && threadIdx.x == 0 && blockIdx.x % counter_rows == 0) counters[blockIdx.x / counter_rows] = 0;
    if (zero_rows) {
        const int per = (zero_width + SAMP_PARTS - 1) / SAMP_PARTS;
        const int z0 = blockIdx.y * per, z1 = z0 + per < zero_width ? z0 + per : zero_width;
        float* zr = zero_rows + (int64_t)blockIdx.x * zero_stride;
        for (int v = z0 + threadIdx.x; v < z1; v += SAMP_THREADS) zr[v] = 0.f;
    }
    const float* row = logits + (int64_t)blockIdx.x * row_stride;
    int g0, g1;
    part_groups(V, blockIdx.y, &g0, &g1);
    __shared__ double2 l_st[SAMP_WAVES];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    float ref = -INFINITY;                                           // of this wavefront; raw fp32 logit (z is monotone in it)
    double sum = 0.0;
    for (int gb = g0 + wave * 64; gb < g1; gb += SAMP_THREADS * STAT_GPT) {
        float v[STAT_GPT][4];
        const int n_u = round_groups<STAT_GPT>(gb, g1);
        // what lies beyond the range comes out as another entry of it: nothing for the maximum, and taken out before the sums below
        load_round<VEC, STAT_GPT>(row, gb, g1, V, v);
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < STAT_GPT; ++u) {
            asm("v_maximum3_f32 %0, %1, %2, %0" : "+v"(mx) : "v"(v[u][0]), "v"(v[u][1]));        // NaN as soon as one of the three is
            asm("v_maximum3_f32 %0, %1, %2, %0" : "+v"(mx) : "v"(v[u][2]), "v"(v[u][3]));
        }
        // A NaN is left out, as below.  By comparisons and only where there is one: v_max3_f32 would leave out quiet ones, but lose what
        // stands beside a signalling one.
        if (__builtin_amdgcn_ballot_w64(mx != mx) != 0) {
            mx = -INFINITY;
#pragma unroll
            for (int u = 0; u < STAT_GPT; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) mx = v[u][j] > mx ? v[u][j] : mx;
        }
        mx = wave_max(mx);
        if (mx > ref) {                                              // wavefront-uniform
            if (ref > -INFINITY) sum *= exp_sum(((double)ref - (double)mx) * rT);
            ref = mx;
        }
        if (ref == -INFINITY) continue;
        const double m = (double)ref;
        auto add = [&](int u) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float l = v[u][j];
                sum += exp_sum(((double)l - m) * rT);                 // the difference is exact: the largest term is exactly 1
            }
        };
        const bool whole = gb + (n_u - 1) * SAMP_THREADS + 63 < g1 && (VEC || 4 * (gb + (n_u - 1) * SAMP_THREADS + 64) <= V);
        if (!whole) {                                                // wavefront-uniform; groups before the last are whole
#pragma unroll
            for (int u = 0; u < STAT_GPT; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int g = gb + u * SAMP_THREADS + lane;
                    if (!(g < g1 && 4 * g + j < V)) v[u][j] = -INFINITY;
                }
        }
#pragma unroll
        for (int u = 0; u < STAT_GPT; ++u) {
            if (u >= n_u) break;
            add(u);
        }
    }
    // fixed order: butterfly inside a wavefront, then over the wavefronts
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) l_st[wave] = make_double2((double)ref, sum);
    __syncthreads();
    if (wave == 0) {
        const double2 c = l_st[lane & (SAMP_WAVES - 1)];
        double2 st = merge_stats<SAMP_WAVES>(c, rT);
        if (st.x == INFINITY) st.y = 0.0;                            // no distribution (see row_stat)
        if (lane == 0) stats[(int64_t)blockIdx.x * SAMP_PARTS + blockIdx.y] = st;
    }
}

__device__ inline void argmax_merge(double& key, int& v, double key2, int v2)
{
    if (key2 > key || (key2 == key && v2 >= 0 && (v < 0 || v2 < v))) { key = key2; v = v2; }
}

__device__ inline void block_argmax(double& key, int& v, double* lk, int* lv)
{
    for (int off = 32; off > 0; off >>= 1) {
        double k2 = __shfl_xor(key, off);
        int v2 = __shfl_xor(v, off);
        argmax_merge(key, v, k2, v2);
    }
    int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) { lk[wave] = key; lv[wave] = v; }
    __syncthreads();
    key = lk[0]; v = lv[0];
    for (int w = 1; w < SAMP_WAVES; ++w) argmax_merge(key, v, lk[w], lv[w]);
}

// 1 / (-ln u) in fp32, u = ((word >> 9) + 0.5) 2^-23.  The logarithm instruction keeps its relative accuracy next to u = 1, where
// the winners of a race are: the largest relative error over all 2^23 words is 2.3e-7 (compared with fp64).
__device__ inline float race_scale(uint32_t word)
{
    const float u = ((float)(word >> 9) + 0.5f) * (1.0f / 8388608.0f);      // exact
    return __builtin_amdgcn_rcpf(-0.69314718f * __builtin_amdgcn_logf(u));
}

// Weights of a race over one row: RACE_PLAIN p; RACE_RES max(0, p - q); RACE_HOT p except 0 at the token `hot` (the residual
// of a one-hot draft distribution).  race_key: the exact key of entry v, fp64, -1 where the weight is not positive.
constexpr int RACE_PLAIN = 0, RACE_RES = 1, RACE_HOT = 2;
constexpr double RACE_SOME = -0.5;            // in the place of a best key: nothing was found, but an entry below `reach` may have a positive weight
struct RaceRow {                              // one race: the row, its largest logit / T and sum, the random stream
    const float *l, *q;
    int V, hot;
    double T, m, S;
    uint32_t k0, k1, c1, c2, c3;
};
template <int KIND>
__device__ inline double race_key(const RaceRow& r, int v)
{
    const double pv = exp((double)r.l[v] / r.T - r.m) / r.S;
    if (!(pv > 0.0)) return -1.0;
    const double w = KIND == RACE_RES ? fmax(0.0, pv - (double)r.q[v]) : (KIND == RACE_HOT && v == r.hot ? 0.0 : pv);
    if (!(w > 0.0)) return -1.0;
    const Philox4 x = philox4x32_10((uint32_t)(v >> 2), r.c1, r.c2, r.c3, r.k0, r.k1);
    const uint32_t word = (v & 2) ? ((v & 1) ? x.w : x.z) : ((v & 1) ? x.y : x.x);
    const double u = ((double)(word >> 9) + 0.5) * (1.0 / 8388608.0);
    return w / (-log(u));
}

// One round of a race, SAMP_GPT groups per lane: keeps in `best` / `best_v` the exact winner among the lane's entries that may win.
// reach: the largest lower bound of a key that this wavefront has met, or that is known or supposed of the row.  A race starts from a
// bound of the whole row: without one a wavefront that holds only keys below the fp32 range's end would evaluate all of them, and with
// peaked logits (a largest logit of 25 over a spread of 2 at T = 0.2) that is nearly every wavefront.  Draw of 256 rows, V = 128256, such
// logits, no bound / a bound: rejected explicit draft 455 / 216 us a call, one-hot 438 / 194, mapped draw of 32000 137 / 86.
// The exponent (l - mx) log2(e) / T, mx the row's largest logit, carries three fp32 roundings (RaceExponent): 126 * 3 * 2^-24 = 2.3e-5 at most
// where the exponential is a normal number, so the fp32 probability is off by less than RACE_EPS of itself, the scale of
// race_scale included.  Below that it counts as 0 with an upper bound of RACE_TINY: such an entry matters only if nothing clear of
// the fp32 range's end competes (RACE_FLOOR, some way above RACE_TINY times the largest scale, 1.7e7), and `reach` is never below that.
constexpr float RACE_EPS = 4.0e-5f, RACE_TINY = 1.2e-38f, RACE_FLOOR = 1.0e-30f;

// log2 of an entry's probability times S: (l c - mx c) * (log2(e) / (T c)), the first term one fused instruction.  c is a power of two
// (1 for the usual temperatures) that keeps every term inside fp32's range for every T > 0, infinite and subnormal ones too:
//   T > 1: 1/2 - l - mx may be twice the largest number, and e.g. T = 1e38 would still give it weight;
//   T < 1e-37: 2^24 - log2(e) / T may be infinite (and 0 times it no number).  With |mx| >= 2^100 c stays 1 and that factor is held at the
//   largest number: two logits that differ do so by 2^77 there, so the product is 0 or far below the range all the same.
struct RaceExponent {
    float c, mc, r;
    __device__ RaceExponent(float mx, double rT)
    {
        const int e = rT < 1.0 ? -1 : (rT > 1e37 && fabsf(mx) < 1.2676506e30f ? 24 : 0);
        c = ldexpf(1.0f, e);
        mc = mx * c;
        r = (float)fmin(ldexp(1.4426950408889634 * rT, -e), 3.4028234663852886e38);
    }
    __device__ float operator()(float l) const { return __builtin_fmaf(l, c, -mc) * r; }
};

template <int KIND>
__device__ inline void race_round(const RaceRow& row, const float (&l)[SAMP_GPT][4], const float (&qv)[SAMP_GPT][4], int gb, int g1, int n_u,
                                  const RaceExponent& exponent, float rS, float& reach, double& best, int& best_v)
{
    const int lane = threadIdx.x & 63;
    const float reach0 = reach;
    float key[SAMP_GPT][4];                                          // the residual races': upper bounds; the plain race's: the fp32 keys
    float lo_max = 0.f;
#pragma unroll
    for (int u = 0; u < SAMP_GPT; ++u) {
#pragma unroll
        for (int j = 0; j < 4; ++j) key[u][j] = -1.f;
        if (u < n_u) {
            const int g = gb + u * SAMP_THREADS + lane;
            const Philox4 x = philox4x32_10((uint32_t)g, row.c1, row.c2, row.c3, row.k0, row.k1);
            const uint32_t word[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float p = __builtin_amdgcn_exp2f(exponent(l[u][j])) * rS;              // 0 for -inf; NaN is never kept
                const float r = race_scale(word[j]);
                if constexpr (KIND == RACE_PLAIN) {
                    key[u][j] = l[u][j] > -INFINITY ? p * r : -1.f;
                    lo_max = fmaxf(lo_max, key[u][j]);
                } else {
                    const float e = p * RACE_EPS + RACE_TINY;
                    const float w = KIND == RACE_RES ? p - qv[u][j] : (4 * g + j == row.hot ? -1.f : p);
                    lo_max = fmaxf(lo_max, (w - e) * r);
                    key[u][j] = l[u][j] > -INFINITY ? (w + e) * r : -1.f;
                }
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) lo_max = fmaxf(lo_max, __shfl_xor(lo_max, off));
    reach = fmaxf(reach, lo_max);
    const float bar = reach * (1.0f - (KIND == RACE_PLAIN ? 3.0f : 1.0f) * RACE_EPS);
    unsigned int may_win = 0;
#pragma unroll
    for (int u = 0; u < SAMP_GPT; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) may_win |= key[u][j] >= bar ? 1u << (4 * u + j) : 0u;
    // a handful of lanes of a wavefront: the entries are read again (and their random words drawn again) rather than kept
    while (may_win) {
        const int at = __builtin_ctz(may_win);
        may_win &= may_win - 1;
        const int v = 4 * (gb + (at >> 2) * SAMP_THREADS + lane) + (at & 3);
        const double k = race_key<KIND>(row, v);
        argmax_merge(best, best_v, k, k > 0.0 ? v : -1);
    }
    if (KIND != RACE_PLAIN && reach == reach0) {
        bool some = false;
#pragma unroll
        for (int u = 0; u < SAMP_GPT; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) some |= key[u][j] >= 0.f;
        if (some) best = fmax(best, RACE_SOME);
    }
}

// Exponential race over the groups [g0, g1) of one row, all SAMP_THREADS threads; every lane's best entry.  No key below `reach` (at
// least RACE_FLOOR) is certain to be found: where the row's best turns out to lie below, the caller looks at all entries.
template <int KIND, bool VEC>
__device__ inline void race_scan(const RaceRow& row, const RaceExponent& exponent, float rS, int g0, int g1, float reach, double& best, int& best_v)
{
    const int wave = threadIdx.x >> 6;
    for (int gb = g0 + wave * 64; gb < g1; gb += SAMP_THREADS * SAMP_GPT) {
        float l[SAMP_GPT][4], qv[SAMP_GPT][4];
        load_round<VEC>(row.l, gb, g1, row.V, -INFINITY, l);
        if (KIND == RACE_RES) load_round<VEC>(row.q, gb, g1, row.V, 0.f, qv);
        race_round<KIND>(row, l, qv, gb, g1, round_groups<SAMP_GPT>(gb, g1), exponent, rS, reach, best, best_v);
    }
}

// a key that the plain race over a row of sum S surely holds: the entry with the largest p, 1 / S, has one of at least 1 / (17 S), as
// -ln u is at most 16.7
__device__ inline float race_known(float rS) { return rS * (1.0f / 17.0f); }

// what a range's workgroup hands to the merge: its best (key, token) of the race
struct RacePart { double key; int64_t v; };

// A workgroup hands in its range's result (thread 0's key and v) and learns whether it is the last of its sequence; if so, every
// thread gets the best over all ranges, in range order (they ascend in token id: an equal key never replaces an earlier one).
// The results go through agent-scope stores and loads, which pass the L2s of the dies by; a fence in their place would write back
// everything this die's L2 holds, once per workgroup (measured: 272 us instead of 98 for the draft's scan at B = 256).
__device__ inline bool merge_parts(RacePart* parts, int part, int32_t* counter, double& key, int& v, int* s_flag)
{
    if (threadIdx.x == 0) {
        __hip_atomic_store((int64_t*)&parts[part].key, __double_as_longlong(key), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&parts[part].v, (int64_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // both stores have arrived before the count says so
        *s_flag = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == SAMP_PARTS - 1;
    }
    __syncthreads();
    if (!*s_flag) return false;
    double k[SAMP_PARTS];
    int t[SAMP_PARTS];
#pragma unroll
    for (int i = 0; i < SAMP_PARTS; ++i) {
        k[i] = __longlong_as_double(__hip_atomic_load((int64_t*)&parts[i].key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        t[i] = (int)__hip_atomic_load(&parts[i].v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    key = -1.0;
    v = -1;
#pragma unroll
    for (int i = 0; i < SAMP_PARTS; ++i) argmax_merge(key, v, k[i], t[i]);
    return true;
}

// Bound by its vector instructions: a Philox block per 4 entries, a logarithm, an exponential and a reciprocal in fp32 per entry
// (58 instructions, about 70 us of issue at B = 256, k = 3, V = 128256 where the two rows' reads would take 45).  Measured there: 76-84 us, 345 us with
// every key in fp64, the accept tests one after the other and the merge in a launch of its own.
template <bool VEC>
__global__ __launch_bounds__(SAMP_THREADS, 4) void reject_scan_kernel(
    int k, int V, const float* __restrict__ logits, const float* __restrict__ q, const int32_t* __restrict__ draft,
    double T, double rT, uint32_t seed_lo, uint32_t seed_hi, uint32_t step4, const double2* __restrict__ stats,
    RacePart* __restrict__ parts, int32_t* __restrict__ counters, int32_t* __restrict__ accept_len, int32_t* __restrict__ out_tokens,
    float* __restrict__ dbg)
{
    const int b = blockIdx.x, part = blockIdx.y;
    const float* L = logits + (int64_t)b * (k + 1) * V;
    const float* Qb = q ? q + (int64_t)b * k * V : nullptr;
    __shared__ int s_n, s_last;
    __shared__ double2 s_st[SPEC_MAX_DRAFT + 1];
    __shared__ double s_m[SPEC_MAX_DRAFT + 1];                        // largest logit / T
    __shared__ double lk[SAMP_WAVES];
    __shared__ int lv[SAMP_WAVES];

    if (threadIdx.x < 64) {
        // the accept tests of the k drafts, one lane each; n = drafts before the first that fails
        const int i = threadIdx.x;
        bool ok = false;
        double P = 0.0, Q = 0.0, u = 0.0;
        for (int r = i / SAMP_PARTS; r < (k + SAMP_PARTS) / SAMP_PARTS * SAMP_PARTS; r += 64 / SAMP_PARTS) {     // the same trips for all lanes
            const double2 st = row_stat(stats, (int64_t)b * (k + 1) + (r <= k ? r : k), rT);
            if (r <= k && i % SAMP_PARTS == 0) { s_st[r] = st; s_m[r] = st.x / T; }
        }
        __builtin_amdgcn_wave_barrier();
        if (i <= k) {
            const int x = i < k ? draft[(int64_t)b * k + i] : -1;
            const bool probe = x >= 0 && x < V;
            const float lx = probe ? L[(int64_t)i * V + x] : 0.f;
            Q = probe ? (Qb ? (double)Qb[(int64_t)i * V + x] : 1.0) : 0.0;      // no q array: one-hot drafts (a deterministic drafter)
            const double2 st = s_st[i];
            const double m = s_m[i];
            if (probe) {
                P = exp((double)lx / T - m) / st.y;
                const Philox4 r = philox4x32_10(0u, (uint32_t)i, (uint32_t)b, step4 + 0u, seed_lo, seed_hi);
                u = (double)(r.x >> 8) * (1.0 / 16777216.0);
                ok = u * Q < P;
            }
            if (dbg && part == 0 && i < k) {
                float* d = dbg + ((int64_t)b * k + i) * 3;
                d[0] = d[1] = d[2] = NAN;
            }
            if (!probe) u = -1.0;
        }
        const unsigned long long pass = __builtin_amdgcn_ballot_w64(ok);
        const int n = __builtin_ctzll(~pass);
        if (dbg && part == 0 && i < k && i <= n && u >= 0.0) {
            float* d = dbg + ((int64_t)b * k + i) * 3;
            d[0] = (float)P; d[1] = (float)Q; d[2] = (float)u;
        }
        if (i == 0) s_n = n;
    }
    __syncthreads();
    const int n = __builtin_amdgcn_readfirstlane(s_n);
    const double2 st = make_double2(uniform(s_st[n].x), uniform(s_st[n].y));
    const float* lrow = L + (int64_t)n * V;
    int g0, g1;
    part_groups(V, part, &g0, &g1);
    double best = -1.0;
    int best_v = -1;
    RaceRow row = {lrow, Qb ? Qb + (int64_t)n * V : nullptr, V, n < k && !Qb ? draft[(int64_t)b * k + n] : -1, T, uniform(s_m[n]), st.y,
                   seed_lo, seed_hi, (uint32_t)n, (uint32_t)b, step4 + 1u};
    const RaceExponent exponent((float)st.x, rT);
    const float rS = __builtin_amdgcn_rcpf((float)st.y);
    // The residual races have no entry that is sure to have a large key, but a draft is rejected where q exceeds p by at least 2^-24 q, and
    // a q of sum 1 leaves as much residual elsewhere: keys above RACE_FLOOR are to be expected.
    if (n < k && Qb) race_scan<RACE_RES, VEC>(row, exponent, rS, g0, g1, RACE_FLOOR, best, best_v);
    else if (n < k) race_scan<RACE_HOT, VEC>(row, exponent, rS, g0, g1, RACE_FLOOR, best, best_v);
    else race_scan<RACE_PLAIN, VEC>(row, exponent, rS, g0, g1, race_known(rS), best, best_v);
    block_argmax(best, best_v, lk, lv);
    if (!merge_parts(parts + (int64_t)b * SAMP_PARTS, part, counters + b, best, best_v, &s_last)) return;
    if (n < k && best >= RACE_SOME && best < (double)RACE_FLOOR) {
        // there are none, but smaller ones: every entry of the row in fp64 (a q that left nothing but such weights: 395 us a call of
        // 64 rows, 75 otherwise)
        for (int v = threadIdx.x; v < V; v += SAMP_THREADS) {
            const double key = Qb ? race_key<RACE_RES>(row, v) : race_key<RACE_HOT>(row, v);
            argmax_merge(best, best_v, key, key > 0.0 ? v : -1);
        }
        block_argmax(best, best_v, lk, lv);
    }
    if (n < k && best_v < 0) {
        // the residual is identically zero: the token comes from the plain race over the whole row
        race_scan<RACE_PLAIN, VEC>(row, exponent, rS, 0, (V + 3) >> 2, race_known(rS), best, best_v);
        block_argmax(best, best_v, lk, lv);
    }
    if (threadIdx.x == 0) accept_len[b] = n;
    for (int i = threadIdx.x; i <= k; i += SAMP_THREADS) out_tokens[(int64_t)b * (k + 1) + i] = i < n ? draft[(int64_t)b * k + i] : (i == n ? best_v : -1);
}

// The draft model's own draw, over the same SAMP_PARTS vocabulary ranges as the verifier's: q = softmax(logits / T)
// written out for the verifier (rounded to fp32 from the fp64 value), and x = argmax_v q_v / (-ln u_v) on random
// stream 2.  row_stats_kernel gives the ranges' statistics; draft_scan_kernel (workgroup = sequence, range) merges them,
// writes its range of q and finds its range's best key; the workgroup that finishes a sequence last picks the token.
// Bound as reject_scan_kernel, with an fp64 exponential more per entry.  With its statistics the draw takes 125-130 us at B = 256,
// V = 128256 (335 before) and 40-43 us at B = 64 (87 before).
template <bool VEC, bool MAPPED>
__global__ __launch_bounds__(SAMP_THREADS, 4) void draft_scan_kernel(
    int V, const float* __restrict__ logits, int64_t logits_stride, double T, double rT, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t step4, uint32_t row, const double2* __restrict__ stats, float* __restrict__ q, int64_t q_stride,
    RacePart* __restrict__ parts, int32_t* __restrict__ counters, int32_t* __restrict__ tok_a, int stride_a, int32_t* __restrict__ tok_b,
    int stride_b, const int32_t* __restrict__ token_map, int q_width)
{
    const int b = blockIdx.x, part = blockIdx.y;
    const float* lrow = logits + (int64_t)b * logits_stride;
    float* qrow = q + (int64_t)b * q_stride;
    __shared__ double lk[SAMP_WAVES];
    __shared__ int lv[SAMP_WAVES];
    __shared__ int s_last;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double2 st = row_stat(stats, b, rT);
    const double m = uniform(st.x), S = uniform(st.y);
    const double rS = S > 0.0 ? 1.0 / S : NAN;                      // without a distribution q is NaN, and the verifier rejects the -1 drawn from it
    const RaceExponent exponent((float)m, rT);
    const float rS32 = (float)rS;
    float reach = race_known(rS32);
    const float known = reach;
    int g0, g1;
    part_groups(V, part, &g0, &g1);
    double best = -1.0;
    int best_v = -1;
    const float none[SAMP_GPT][4] = {};
    const RaceRow race = {lrow, nullptr, V, -1, T, m / T, S, seed_lo, seed_hi, row, (uint32_t)b, step4 + 2u};
    for (int gb = g0 + wave * 64; gb < g1; gb += SAMP_THREADS * SAMP_GPT) {
        float l[SAMP_GPT][4];
        const int n_u = round_groups<SAMP_GPT>(gb, g1);
        load_round<VEC>(lrow, gb, g1, V, -INFINITY, l);
#pragma unroll
        for (int u = 0; u < SAMP_GPT; ++u) {
            if (u >= n_u) break;
            const int g = gb + u * SAMP_THREADS + lane;
            float p[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double x = ((double)l[u][j] - m) * rT;
                const float pj = (float)(exp_sum(x) * rS);
                p[j] = x == x ? pj : NAN;                           // a NaN logit (and -inf at an infinite T)
            }
            if (g < g1) {
                if constexpr (VEC && !MAPPED) {
                    *(float4*)(qrow + 4 * (int64_t)g) = make_float4(p[0], p[1], p[2], p[3]);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int v = 4 * g + j;
                        if (v >= V) continue;
                        const int at = MAPPED ? token_map[v] : v;                               // (a mapped row was cleared by the statistics kernel)
                        if (MAPPED && (unsigned)at >= (unsigned)q_width) l[u][j] = -INFINITY;    // outside the target's vocabulary: never written, never drawn
                        else qrow[at] = p[j];
                    }
                }
            }
        }
        race_round<RACE_PLAIN>(race, l, none, gb, g1, n_u, exponent, rS32, reach, best, best_v);
    }
    block_argmax(best, best_v, lk, lv);
    if (!merge_parts(parts + (int64_t)b * SAMP_PARTS, part, counters + b, best, best_v, &s_last)) return;
    if (MAPPED && S > 0.0 && best < (double)known) {
        // a map may leave out the most probable entry, and then there may be no key of that size: every entry of the row in fp64
        for (int v = threadIdx.x; v < V; v += SAMP_THREADS) {
            if ((unsigned)token_map[v] >= (unsigned)q_width) continue;
            const double key = race_key<RACE_PLAIN>(race, v);
            argmax_merge(best, best_v, key, key > 0.0 ? v : -1);
        }
        block_argmax(best, best_v, lk, lv);
    }
    if (threadIdx.x == 0) {
        if (MAPPED && best_v >= 0) best_v = token_map[best_v];
        if (tok_a) tok_a[(int64_t)b * stride_a] = best_v;
        if (tok_b) tok_b[(int64_t)b * stride_b] = best_v;
    }
}

}  // namespace specv

// workspace: the ranges' row statistics [B * (k + 1)][SAMP_PARTS] double2, the ranges' race results [B][SAMP_PARTS], then the
// sequences' arrival counters [B]
static size_t sample_stats_bytes(int64_t rows) { return specv::align_up((size_t)rows * specv::SAMP_PARTS * sizeof(double2), 256); }
static size_t sample_parts_bytes(int64_t B) { return specv::align_up((size_t)B * specv::SAMP_PARTS * sizeof(specv::RacePart), 256); }

extern "C" size_t spec_sample_workspace_bytes(int32_t B, int32_t k)
{
    if (B < 1 || k < 0) return 0;
    return sample_stats_bytes((int64_t)B * (k + 1)) + sample_parts_bytes(B) + specv::align_up((size_t)B * sizeof(int32_t), 256);
}

namespace specv {

// argument checks and the launches shared by both entry points; ws: spec_sample_workspace_bytes(B, k) bytes of device memory
static spec_status reject_sample_launch(const char* who, int32_t B, int32_t k, int32_t V, const float* dev_logits, const float* dev_q,
                                        const int32_t* dev_draft_tokens, float temperature, uint64_t seed, uint64_t step,
                                        int32_t* dev_accept_len, int32_t* dev_out_tokens, float* dev_dbg, void* ws, hipStream_t s)
{
    double2* stats = (double2*)ws;
    if (B < 1 || k < 0 || k > SPEC_MAX_DRAFT || V < 1) { set_error("%s: B, k or V out of range", who); return SPEC_EINVAL; }
    if (!(temperature > 0.f)) { set_error("%s: temperature must be > 0", who); return SPEC_EINVAL; }
    if (step >= (1ull << 30)) { set_error("%s: step must be < 2^30", who); return SPEC_EINVAL; }
    if (!dev_logits || !dev_accept_len || !dev_out_tokens || !ws || (k > 0 && !dev_draft_tokens)) {
        set_error("%s: null pointer", who); return SPEC_EINVAL;
    }
    const double T = (double)temperature, rT = 1.0 / T;
    RacePart* parts = (RacePart*)((char*)ws + sample_stats_bytes((int64_t)B * (k + 1)));
    int32_t* counters = (int32_t*)((char*)parts + sample_parts_bytes(B));
    prof_mark(PC_OTHER, s);
    const bool vec = rows_vec(dev_logits, V, V) && (!dev_q || rows_vec(dev_q, V, V));
    const dim3 stat_grid((unsigned)(B * (k + 1)), SAMP_PARTS), grid((unsigned)B, SAMP_PARTS);
#define SPEC_REJECT_LAUNCH(VECV) do { \
        row_stats_kernel<VECV><<<stat_grid, SAMP_THREADS, 0, s>>>(dev_logits, (int64_t)V, V, rT, stats, counters, k + 1); \
        SPEC_LAUNCH_CHECK("row_stats_kernel"); \
        prof_mark(PC_SAMPLE_STATS, s); \
        reject_scan_kernel<VECV><<<grid, SAMP_THREADS, 0, s>>>(k, V, dev_logits, dev_q, dev_draft_tokens, T, rT, (uint32_t)seed, (uint32_t)(seed >> 32), \
                                                              (uint32_t)(step * 4u), stats, parts, counters, dev_accept_len, dev_out_tokens, dev_dbg); \
    } while (0)
    if (vec) SPEC_REJECT_LAUNCH(true); else SPEC_REJECT_LAUNCH(false);
#undef SPEC_REJECT_LAUNCH
    SPEC_LAUNCH_CHECK("reject_scan_kernel");
    prof_mark(PC_SAMPLE_DRAW, s);
    return SPEC_OK;
}

// Workspace of spec_reject_sample_static: device memory that exists from the moment the library is loaded, so
// that entry point never allocates.  Every GPU holds its own copy at its own address; the array's name is only a
// host-side handle, the address kernels are given comes from hipGetSymbolAddress with that GPU current.
constexpr int SAMP_STATIC_ROWS = 4096;                  // B * (k + 1) at most: 512 KiB of row statistics, as much for race results and 16 KiB of counters (sized for k = 0, B = 4096) per GPU
constexpr size_t SAMP_STATIC_BYTES = (size_t)SAMP_STATIC_ROWS * (SAMP_PARTS * (sizeof(double2) + sizeof(RacePart)) + sizeof(int32_t)) + 768;
static __device__ __align__(256) unsigned char scratch[SAMP_STATIC_BYTES];
constexpr int SAMP_MAX_DEVICES = 64;
static void* g_scratch_ptr[SAMP_MAX_DEVICES];
static std::mutex g_scratch_mutex;

static spec_status static_scratch(void** out)
{
    int dev = -1;
    SPEC_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= SAMP_MAX_DEVICES) { set_error("spec_reject_sample_static: device index %d is beyond %d", dev, SAMP_MAX_DEVICES - 1); return SPEC_EUNSUPPORTED; }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) { set_error("spec_reject_sample_static: hipGetSymbolAddress failed: %s", hipGetErrorString(e)); return SPEC_EHIP; }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SPEC_OK;
}

}  // namespace specv

extern "C" spec_status spec_reject_sample(int32_t B, int32_t k, int32_t V, const float* dev_logits, const float* dev_q,
                                          const int32_t* dev_draft_tokens, float temperature, uint64_t seed,
                                          uint64_t step, int32_t* dev_accept_len, int32_t* dev_out_tokens,
                                          float* dev_dbg, void* dev_workspace, size_t workspace_bytes, void* stream)
{
    using namespace specv;
    if (B >= 1 && k >= 0 && dev_workspace && workspace_bytes < spec_sample_workspace_bytes(B, k)) { set_error("spec_reject_sample: workspace too small"); return SPEC_EINVAL; }
    return reject_sample_launch("spec_reject_sample", B, k, V, dev_logits, dev_q, dev_draft_tokens, temperature, seed, step, dev_accept_len,
                                dev_out_tokens, dev_dbg, dev_workspace, (hipStream_t)stream);
}

extern "C" spec_status spec_reject_sample_static(int32_t B, int32_t k, int32_t V, const float* dev_logits, const float* dev_q,
                                                 const int32_t* dev_draft_tokens, float temperature, uint64_t seed,
                                                 uint64_t step, int32_t* dev_accept_len, int32_t* dev_out_tokens,
                                                 float* dev_dbg, void* stream)
{
    using namespace specv;
    if (B >= 1 && k >= 0 && k <= SPEC_MAX_DRAFT && (int64_t)B * (k + 1) > SAMP_STATIC_ROWS) {
        set_error("spec_reject_sample_static: B * (k + 1) = %lld rows exceed the built-in scratch of %d rows (use spec_reject_sample with a workspace)",
                  (long long)B * (k + 1), SAMP_STATIC_ROWS);
        return SPEC_EINVAL;
    }
    void* stats = nullptr;
    spec_status st = static_scratch(&stats);
    if (st != SPEC_OK) return st;
    return reject_sample_launch("spec_reject_sample_static", B, k, V, dev_logits, dev_q, dev_draft_tokens, temperature, seed, step,
                                dev_accept_len, dev_out_tokens, dev_dbg, stats, (hipStream_t)stream);
}

extern "C" size_t spec_draft_sample_workspace_bytes(int32_t B)
{
    if (B < 1) return 0;
    return sample_stats_bytes(B) + sample_parts_bytes(B) + specv::align_up((size_t)B * sizeof(int32_t), 256);
}

static spec_status draft_sample_launch(const char* who, int32_t B, int32_t V, const float* dev_logits, int64_t logits_row_stride,
                                       float temperature, uint64_t seed, uint64_t step, int32_t row,
                                       int32_t* dev_tokens_a, int32_t stride_a, int32_t* dev_tokens_b, int32_t stride_b,
                                       float* dev_q, int64_t q_row_stride, const int32_t* dev_token_map, int32_t q_width,
                                       void* dev_workspace, size_t workspace_bytes, void* stream)
{
    using namespace specv;
    if (B < 1 || V < 1 || row < 0 || row > SPEC_MAX_DRAFT) { set_error("%s: B, V or row out of range", who); return SPEC_EINVAL; }
    if (!(temperature > 0.f)) { set_error("%s: temperature must be > 0", who); return SPEC_EINVAL; }
    if (step >= (1ull << 30)) { set_error("%s: step must be < 2^30", who); return SPEC_EINVAL; }
    if (!dev_logits || !dev_q || (!dev_tokens_a && !dev_tokens_b)) { set_error("%s: null pointer", who); return SPEC_EINVAL; }
    if (logits_row_stride < V || q_row_stride < q_width || (dev_tokens_a && stride_a < 1) || (dev_tokens_b && stride_b < 1)) {
        set_error("%s: a row stride is smaller than the row", who); return SPEC_EINVAL;
    }
    if (!dev_workspace || workspace_bytes < spec_draft_sample_workspace_bytes(B)) { set_error("%s: workspace missing or too small", who); return SPEC_EINVAL; }
    hipStream_t s = (hipStream_t)stream;
    prof_mark(PC_OTHER, s);
    double2* stats = (double2*)dev_workspace;
    RacePart* parts = (RacePart*)((char*)dev_workspace + sample_stats_bytes(B));
    int32_t* counters = (int32_t*)((char*)parts + sample_parts_bytes(B));
    const double T = (double)temperature, rT = 1.0 / T;
    const bool vec = rows_vec(dev_logits, logits_row_stride, V) && (dev_token_map || rows_vec(dev_q, q_row_stride, V));
    const dim3 grid((unsigned)B, SAMP_PARTS);
#define SPEC_DRAFT_LAUNCH(VECV, MAPV) do { \
        row_stats_kernel<VECV><<<grid, SAMP_THREADS, 0, s>>>(dev_logits, logits_row_stride, V, rT, stats, counters, 1, \
                                                            dev_token_map ? dev_q : nullptr, q_row_stride, q_width); \
        draft_scan_kernel<VECV, MAPV><<<grid, SAMP_THREADS, 0, s>>>(V, dev_logits, logits_row_stride, T, rT, (uint32_t)seed, (uint32_t)(seed >> 32), \
                                                             (uint32_t)(step * 4u), (uint32_t)row, stats, dev_q, q_row_stride, parts, counters, \
                                                             dev_tokens_a, stride_a, dev_tokens_b, stride_b, dev_token_map, dev_token_map ? q_width : V); \
    } while (0)
    if (dev_token_map) { if (vec) SPEC_DRAFT_LAUNCH(true, true); else SPEC_DRAFT_LAUNCH(false, true); }
    else { if (vec) SPEC_DRAFT_LAUNCH(true, false); else SPEC_DRAFT_LAUNCH(false, false); }
#undef SPEC_DRAFT_LAUNCH
    SPEC_LAUNCH_CHECK("draft sampling kernels");
    prof_mark(PC_DRAFT_SAMPLE, s);
    return SPEC_OK;
}

extern "C" spec_status spec_draft_sample(int32_t B, int32_t V, const float* dev_logits, int64_t logits_row_stride,
                                         float temperature, uint64_t seed, uint64_t step, int32_t row,
                                         int32_t* dev_tokens_a, int32_t stride_a, int32_t* dev_tokens_b, int32_t stride_b,
                                         float* dev_q, int64_t q_row_stride, void* dev_workspace, size_t workspace_bytes, void* stream)
{
    return draft_sample_launch("spec_draft_sample", B, V, dev_logits, logits_row_stride, temperature, seed, step, row, dev_tokens_a, stride_a,
                               dev_tokens_b, stride_b, dev_q, q_row_stride, nullptr, V, dev_workspace, workspace_bytes, stream);
}

extern "C" spec_status spec_draft_sample_mapped(int32_t B, int32_t V_d, const float* dev_logits, int64_t logits_row_stride,
                                                float temperature, uint64_t seed, uint64_t step, int32_t row,
                                                int32_t* dev_tokens_a, int32_t stride_a, int32_t* dev_tokens_b, int32_t stride_b,
                                                float* dev_q, int64_t q_row_stride, const int32_t* dev_token_map, int32_t V_full,
                                                void* dev_workspace, size_t workspace_bytes, void* stream)
{
    if (!dev_token_map || V_full < V_d) { specv::set_error("spec_draft_sample_mapped: no token map, or V_full below V_d"); return SPEC_EINVAL; }
    return draft_sample_launch("spec_draft_sample_mapped", B, V_d, dev_logits, logits_row_stride, temperature, seed, step, row, dev_tokens_a,
                               stride_a, dev_tokens_b, stride_b, dev_q, q_row_stride, dev_token_map, V_full, dev_workspace, workspace_bytes, stream);
}

namespace specv {

// pending[b] = (tokens[b][n_b], out[b][n_b]) and tokens[b][0] = out[b][n_b]: the inputs of the next step
__global__ void next_inputs_kernel(int B, int k, int32_t* __restrict__ tokens, const int32_t* __restrict__ out_tokens,
                                   const int32_t* __restrict__ accept_len, int32_t* __restrict__ pending)
{
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    int n = accept_len[b];
    n = n < 0 ? 0 : (n > k ? k : n);
    int32_t last_input = tokens[(int64_t)b * (k + 1) + n];
    int32_t emitted = out_tokens[(int64_t)b * (k + 1) + n];
    if (pending) { pending[2 * b] = last_input; pending[2 * b + 1] = emitted; }
    tokens[(int64_t)b * (k + 1)] = emitted;
}

}  // namespace specv

namespace specv {

// pending_hidden[b] = (H[b][n-1] or its own old row 1 if n = 0, H[b][n]); workgroup = (batch entry, 1024 channels)
__global__ void next_hidden_kernel(int k, int d, const float* __restrict__ target_hidden, const int32_t* __restrict__ accept_len,
                                   float* __restrict__ pending_hidden)
{
    const int b = blockIdx.x;
    int n = accept_len[b];
    n = n < 0 ? 0 : (n > k ? k : n);
    const float* H = target_hidden + (int64_t)b * (k + 1) * d;
    float* p = pending_hidden + (int64_t)b * 2 * d;
    const int c_end = min(d, (int)(blockIdx.y + 1) * 1024);
    for (int c = blockIdx.y * 1024 + threadIdx.x; c < c_end; c += blockDim.x) {
        const float before_kept = n >= 1 ? H[(int64_t)(n - 1) * d + c] : p[d + c];     // read row 1 before it is overwritten
        const float before_emitted = H[(int64_t)n * d + c];
        p[c] = before_kept;
        p[d + c] = before_emitted;
    }
}

}  // namespace specv

extern "C" spec_status spec_next_step_hidden(int32_t B, int32_t k, int32_t d, const float* dev_target_hidden,
                                             const int32_t* dev_accept_len, float* dev_pending_hidden, void* stream)
{
    using namespace specv;
    if (B < 1 || k < 0 || k > SPEC_MAX_DRAFT || d < 1) { set_error("spec_next_step_hidden: B, k or d out of range"); return SPEC_EINVAL; }
    if (!dev_target_hidden || !dev_accept_len || !dev_pending_hidden) { set_error("spec_next_step_hidden: null pointer"); return SPEC_EINVAL; }
    next_hidden_kernel<<<dim3((unsigned)B, (unsigned)cdiv(d, 1024)), 256, 0, (hipStream_t)stream>>>(k, d, dev_target_hidden, dev_accept_len, dev_pending_hidden);
    SPEC_LAUNCH_CHECK("next_hidden_kernel");
    return SPEC_OK;
}

extern "C" spec_status spec_next_step_inputs(int32_t B, int32_t k, int32_t* dev_tokens, const int32_t* dev_out_tokens,
                                             const int32_t* dev_accept_len, int32_t* dev_pending, void* stream)
{
    using namespace specv;
    if (B < 1 || k < 0 || k > SPEC_MAX_DRAFT) { set_error("spec_next_step_inputs: B or k out of range"); return SPEC_EINVAL; }
    if (!dev_tokens || !dev_out_tokens || !dev_accept_len) { set_error("spec_next_step_inputs: null pointer"); return SPEC_EINVAL; }
    next_inputs_kernel<<<(unsigned)cdiv(B, 256), 256, 0, (hipStream_t)stream>>>(B, k, dev_tokens, dev_out_tokens, dev_accept_len, dev_pending);
    SPEC_LAUNCH_CHECK("next_inputs_kernel");
    return SPEC_OK;
}
