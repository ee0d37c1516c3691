// SBVR encoding (Algorithm 1 with the bitvector assignment of Sec. 4.2) on
// the GPU: for every 128-weight group, search the coefficient sets of the
// (r, s, b) grid (Eqs. 4-11) for the one with the smallest mean squared error
// of nearest-subset-sum reconstruction, then give each weight the pattern of
// its nearest subset sum.
//
// The arithmetic is the search's definition carried out in binary64 in a
// fixed order, so the result is bit-identical to any implementation that
// follows the same definition (this file is compiled without floating-point
// contraction):
//   - group statistics in element order: min, max, sum; mean = sum / n;
//   - q95: the linearly interpolated 95th percentile of the sorted group,
//     s[lo] + frac * (s[lo+1] - s[lo]) at position 0.95 (n - 1);
//   - S_j = s_min + (j+1) s_gran, s_min = 2 q95, s_max = 1.1 (max - min),
//     s_gran = (s_max - s_min) / N_scale (Eqs. 6, 8, 10, 11);
//     B_k = b_min + k b_gran, b_max = 2 |mean| / K, b_min = -b_max,
//     b_gran = (b_max - b_min) / N_bias (Eqs. 7, 9, 10, 11);
//     R: -1 + (i+1) (0.5 / N_1) for i < N_1, then -2 + i (1 / N_2) for i < N_2;
//   - entry coefficients c_i = fp16((s r^i) / N(r) + b), r^i by repeated
//     multiplication, N(r) = sum_i abs(r^i) accumulated in i order (1 for the
//     literal form of Eq. 4); entries with s <= 0 or a non-finite c are skipped;
//   - subset sums in bit order, nearest = first strict minimum of
//     abs(x - sum_p) over p ascending, MSE = (sum_j (x_j - sum)^2 in j order) / n,
//     best entry = first strict minimum over entries in (r, s, b) order;
//   - no admissible entry: c = (fp16(mean), 0, ...).
//
// The search needs only each element's smallest squared distance to a subset
// sum, min_p fl((x - sum_p)^2), which equals the square of the nearest
// difference (the rounded square is monotone in |d|); the pattern itself is
// found once, for the chosen entry.
//
// Screening.  Scoring an entry by that definition takes 128 x 2^k distances.
// Almost every entry is ruled out much more cheaply: with the subset sums
// sorted (s_0 <= .. <= s_n) and m_p the midpoint of s_(p-1) and s_p,
//     sum_j min_p (x_j - s_p)^2
//         = sum_j (x_j - s_n)^2 - 2 sum_p (s_p - s_(p-1)) g(m_p),
//     g(m) = sum_j max(0, m - x_j),
// and g is one convex function per group.  The group's g is tabulated as
// chords over ENC_CELLS equal cells of its range; a chord lies above g, so the
// table gives a lower bound of an entry's error with one lookup per midpoint
// instead of 128 distances per subset sum (about 300 vector instructions per
// entry at k = 4, against 6144).  The bound is computed in binary32;
// entry_bound() subtracts a bound on its rounding.  Entries whose lower bound exceeds the
// error of an entry already scored can neither win nor tie and are dropped
// (Gaussian groups keep about 5 of 1024); the others are scored in binary64,
// first with the terms added across the lanes, then, where that leaves a
// possible winner (within 2^-40 of the smallest), in the definition's order.
// Every entry that could be the first minimum is scored by the definition, so
// the result does not depend on the screening.
//
// Work split: one wavefront per group.  In the screening lane l takes
// ENC_RUN consecutive entries (neighbouring entries share r and s, so the
// divisions of Eq. 4 are made once per (r, s)); in the scoring every lane takes
// its two elements of one entry.  Where more than ENC_LIST entries of a chunk
// survive (degenerate groups), or more than enc_serial(k) sets are left after
// the first one is scored, lanes take entries instead and the elements run in
// order, so such a group costs about what an unscreened search does.  Grids of
// a few entries are not screened at all (ENC_PLAIN_SUMS).
// Bound: vector instruction issue, about 7600 instructions per group at k = 4,
// of which about 4600 are the (binary32) bounds; 3200 at k = 1.  Measured
// against scoring every entry by the definition (with pruning), 1024 entries,
// N(0, 0.02^2), one value in a thousand at 8 sigma: 4096 x 4096, encoding and
// packing, k = 4 17.9 -> 1.48 ms, with the encoder cache at k = 3 7.6 -> 0.91
// ms; encoding alone at k = 1 3.5 -> 0.75 ms.  Groups whose entries are all
// alike (magnitudes below binary16's) keep every entry: 1024 x 2048, k = 4 3.05
// -> 2.26 ms, k = 1 0.50 -> 0.49.
#include "device_ops.h"
#include "f16_round.h"
#include "launch.h"

#include <climits>

namespace sbvr {

constexpr int ENC_THREADS = 64;  // one wavefront per group

__device__ __forceinline__ double f16_bits_to_double(uint16_t h)
{
    return (double)half_bits_to_float(h);  // both conversions exact
}

// The part of an entry's coefficients that r and s fix, (s r^i) / N(r).
template <int K>
struct EntryShape {
    double q[K];

    __device__ __forceinline__ void set(double r, double s, bool normalise)
    {
        double norm = 1.0;
        if (normalise) {
            double a = 1.0, t = 0.0;
#pragma unroll
            for (int i = 0; i < K; ++i) {
                t += fabs(a);
                a *= r;
            }
            norm = t;
        }
        double pw = 1.0;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            q[i] = (s * pw) / norm;
            pw *= r;
        }
    }

    // the coefficients at bias b; false if one is not finite
    __device__ __forceinline__ bool coeffs(double b, uint16_t *c) const
    {
        bool ok = true;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            c[i] = f64_to_f16_odd(q[i] + b);
            ok = ok && (c[i] & 0x7c00u) != 0x7c00u;
        }
        return ok;
    }
};

template <int K>
__device__ __forceinline__ void subset_sums(const uint16_t *c, double *sums)
{
    double cv[K];
#pragma unroll
    for (int i = 0; i < K; ++i)
        cv[i] = f16_bits_to_double(c[i]);
#pragma unroll
    for (int p = 0; p < (1 << K); ++p) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < K; ++i)
            if ((p >> i) & 1)
                t += cv[i];
        sums[p] = t;
    }
}

// Nearest subset sum of x: pattern index and the signed difference x - sum.
template <int K>
__device__ __forceinline__ int nearest(const double *sums, double x, double &diff)
{
    int best = 0;
    double bd = x - sums[0];
#pragma unroll
    for (int p = 1; p < (1 << K); ++p) {
        const double d = x - sums[p];
        if (fabs(d) < fabs(bd)) {
            bd = d;
            best = p;
        }
    }
    diff = bd;
    return best;
}

// Smallest squared distance from x to a subset sum: the square of the nearest
// difference, without tracking which sum it was (one subtraction and one
// minimum with a magnitude per sum).
template <int K>
__device__ __forceinline__ double nearest_sq(const double *sums, double x)
{
    double m = fabs(x - sums[0]);
#pragma unroll
    for (int p = 1; p < (1 << K); ++p)
        m = fmin(m, fabs(x - sums[p]));
    return m * m;
}

__device__ __forceinline__ double wave_min_f64(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v = fmin(v, __shfl_xor(v, off));
    return v;
}

template <int K>
__device__ __forceinline__ double entry_mse(const double *D, const double *sums)
{
    double err = 0.0;
    for (int j = 0; j < GROUP; ++j) {
        err += nearest_sq<K>(sums, D[j]);
    }
    return err / (double)GROUP;
}

struct EncodeArgs {
    const float *W;
    uint32_t *planes;  // canonical [O][G][K][4]
    uint16_t *coeffs;  // canonical [O][G][K]
    double *mse;       // [O][G] or null
    int O, I;
    int n_ratio1, n_ratio2, n_scale, n_bias, normalise;
};

constexpr int ENC_CELLS = 512;                    // chords of the group's g
constexpr int ENC_RUN = 16;                       // consecutive entries a lane screens
constexpr int ENC_CHUNK = ENC_RUN * ENC_THREADS;  // entries screened at a time
constexpr int ENC_LIST = 32;                      // entries scored across the lanes, at most
// Grids of at most this many subset sums (entries x 2^k) are scored by the
// definition at once: a few rounds of a lane per entry cost less than the table
// and the serial scoring of the survivors.  512 x 1024, N(0, 0.02^2), without
// and with the screening: k = 1, 64 entries 20 / 40 us; k = 2, 32 entries 26 /
// 29; k = 3, 16 entries 36 / 36; above the line k = 2, 64 entries 26 / 29, but
// with the cache (256 x 14336) 1050 / 720; k = 3, 32 entries 36 / 33; k = 4, 16
// entries 47 / 35.
constexpr int ENC_PLAIN_SUMS = 128;
// When more sets than this are left after the first one is scored (groups whose
// entries are nearly alike; at k = 1 most), a lane takes a set and the elements
// run in order (2^k distances each), instead of one set after the other across
// the lanes.  512 x 1024, with up to 32 one after the other and with this: k =
// 1, 1024 entries, N(0, 0.02^2) 106 / 50 us; 32 equal entries 168 / 48 (k = 3),
// 190 / 69 (k = 4).  With 8 at k = 4, ternary weights with the cache (256 x
// 14336) took 1342 instead of 1190.
__host__ __device__ constexpr int enc_serial(int k) { return k == 1 ? 4 : (k == 2 ? 8 : 12); }
// Two orders of adding 128 non-negative binary64 terms differ by less than
// this share of their sum (2 x 127 roundings of 2^-53).
constexpr double ENC_ORDER_EPS = 0x1p-40;
// The screening is off (every entry is kept) where its binary32 sums might
// overflow; coefficients are binary16, so such a group has no close entry.
constexpr float ENC_SCREEN_MAX = 1e15f;

// A wavefront's LDS for one group.
struct EncodeLds {
    double D[GROUP];      // the values in element order (read as broadcasts)
    double E[GROUP + 1];  // table build: twice the sums of the t smallest values; scoring: an
                          // entry's terms in element order
    float2 cell[ENC_CELLS + 2];  // chords (value at 0, slope) in m2 = 2 m; below and above the range
    union {
        float lb[ENC_CHUNK];   // lower bounds, entry of (lane, i) at i * 64 + lane
        int mark[ENC_CELLS];   // table build: values up to and in each cell
    };
    int list[ENC_LIST];
};

// What the search knows about a group besides L (wavefront-uniform).
struct GroupStats {
    double mn, mx, q95;
    float lo2, ih;  // 2 min, cells per unit of 2 x
    float X, S2, T2;  // max |x|, sum x^2, 2 sum x
};

__device__ __forceinline__ float lane_f32(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ double lane_f64(double v, int l)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum over the wavefront (wavefront-uniform, in a tree's order).
__device__ __forceinline__ double wave_sum_f64(double v)
{
    v += dpp_f64<DPP_QUAD_XOR1>(v);
    v += dpp_f64<DPP_QUAD_XOR2>(v);
    v += dpp_f64<DPP_ROW_HALF_MIRROR>(v);
    v += dpp_f64<DPP_ROW_MIRROR>(v);
    return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}

__device__ __forceinline__ float wave_min_f32(float v)
{
    v = fminf(v, dpp_f32<DPP_QUAD_XOR1>(v));
    v = fminf(v, dpp_f32<DPP_QUAD_XOR2>(v));
    v = fminf(v, dpp_f32<DPP_ROW_HALF_MIRROR>(v));
    v = fminf(v, dpp_f32<DPP_ROW_MIRROR>(v));
    return fminf(fminf(lane_f32(v, 0), lane_f32(v, 16)), fminf(lane_f32(v, 32), lane_f32(v, 48)));
}

// binary32 at or above a non-negative binary64 value.
__device__ __forceinline__ float f32_above(double v) { return (float)v * (1.0f + 0x1p-20f); }

// Cell of 2 m: 0 below the range, ENC_CELLS + 1 above it.
__device__ __forceinline__ int cell_of(const GroupStats &t, float m2)
{
    const float u = fmaf(m2 - t.lo2, t.ih, 1.0f);
    return (int)__builtin_amdgcn_fmed3f(u, 0.0f, (float)(ENC_CELLS + 1));
}

// Sorts the group (x0, x1: the lane's two values), takes the order statistics
// and, for a screened search, tabulates g.  With t values below m and P their sum, 2 g(m) = m2 t - 2 P
// for m2 = 2 m.
template <bool SCREENED>
__device__ GroupStats group_table(EncodeLds &L, float x0, float x1)
{
    const int lane = threadIdx.x;
    GroupStats st = {};
    // bitonic sort of 128 values, sorted value 2 lane + h in v[h]; med3 with
    // an infinity is min or max
    float v0 = x0, v1 = x1;
#pragma unroll
    for (int k = 2; k <= GROUP; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j >= 2; j >>= 1) {
            const bool keep_min = ((lane & (j >> 1)) == 0) == ((lane & (k >> 1)) == 0);
            const float sel = keep_min ? -__builtin_inff() : __builtin_inff();
            v0 = __builtin_amdgcn_fmed3f(v0, __shfl_xor(v0, j >> 1), sel);
            v1 = __builtin_amdgcn_fmed3f(v1, __shfl_xor(v1, j >> 1), sel);
        }
        const bool asc = (lane & (k >> 1)) == 0;
        const float a = fminf(v0, v1), b = fmaxf(v0, v1);
        v0 = asc ? a : b;
        v1 = asc ? b : a;
    }
    st.mn = (double)lane_f32(v0, 0);
    st.mx = (double)lane_f32(v1, 63);

    // sorted positions lo and lo+1 of the linear-interpolation percentile
    constexpr double pos = 0.95 * (double)(GROUP - 1);
    constexpr int lo = (int)pos;
    const double frac = pos - (double)lo;
    static_assert(lo % 2 == 0, "both positions in one lane");
    const double q0 = (double)lane_f32(v0, lo / 2), q1 = (double)lane_f32(v1, lo / 2);
    st.q95 = q0 + frac * (q1 - q0);
    if constexpr (!SCREENED) {
        __syncthreads();
        return st;
    }

    // twice the sums of the t smallest values
    double incl = (double)v0 + (double)v1;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double up = __shfl_up(incl, off);
        incl += lane >= off ? up : 0.0;
    }
    double excl = __shfl_up(incl, 1);
    excl = lane > 0 ? excl : 0.0;
    L.E[2 * lane] = 2.0 * excl;
    L.E[2 * lane + 1] = 2.0 * (excl + (double)v0);
    const double total2 = 2.0 * lane_f64(incl, 63);
    if (lane == 63)
        L.E[GROUP] = total2;

    const double range2 = 2.0 * st.mx - 2.0 * st.mn;
    const double inv_h2 = range2 > 0.0 ? (double)ENC_CELLS / range2 : 0.0;
    st.lo2 = 2.0f * (float)st.mn;
    st.ih = range2 > 0.0 ? (float)fmin(inv_h2, 1e38) : 1e38f;
    st.X = (float)fmax(fabs(st.mn), fabs(st.mx));
    st.S2 = (float)wave_sum_f64((double)x0 * (double)x0 + (double)x1 * (double)x1);
    st.T2 = (float)total2;

    // values in and below each cell: the last value of a cell marks it, then
    // a running maximum over the cells
    constexpr int PER = ENC_CELLS / 64;
    static_assert(PER == 8, "two 16-byte stores per lane");
    *(int4 *)&L.mark[PER * lane] = make_int4(0, 0, 0, 0);
    *(int4 *)&L.mark[PER * lane + 4] = make_int4(0, 0, 0, 0);
    __syncthreads();
    auto cell_in = [&](float x) { return min(max(cell_of(st, 2.0f * x) - 1, 0), ENC_CELLS - 1); };
    const int c0 = cell_in(v0), c1 = cell_in(v1), c2 = __shfl_down(c0, 1);
    if (c0 != c1)
        L.mark[c0] = 2 * lane + 1;
    if (lane == 63 || c1 != c2)
        L.mark[c1] = 2 * lane + 2;
    __syncthreads();
    int n[PER];
    *(int4 *)&n[0] = *(const int4 *)&L.mark[PER * lane];
    *(int4 *)&n[4] = *(const int4 *)&L.mark[PER * lane + 4];
#pragma unroll
    for (int i = 1; i < PER; ++i)
        n[i] = max(n[i], n[i - 1]);
    int below = n[PER - 1];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(below, off);
        below = max(below, lane >= off ? up : 0);
    }
    below = __shfl_up(below, 1);
    below = lane > 0 ? below : 0;

    const double h2 = range2 / (double)ENC_CELLS, lo2 = 2.0 * st.mn;
    double u = lo2 + (double)(PER * lane) * h2;
    double g = u * (double)below - L.E[below];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int t = max(below, n[i]);
        const double un = lo2 + (double)(PER * lane + i + 1) * h2;
        const double gn = un * (double)t - L.E[t];
        const double slope = (gn - g) * inv_h2;
        L.cell[1 + PER * lane + i] = make_float2((float)(g - slope * u), (float)slope);
        u = un;
        g = gn;
    }
    if (lane == 0) {
        L.cell[0] = make_float2(0.0f, 0.0f);
        L.cell[ENC_CELLS + 1] = make_float2((float)-total2, (float)GROUP);
    }
    __syncthreads();
    return st;
}

// s[0 .. 2n) sorted from two sorted halves of n (odd-even merge).
template <int N>
__device__ __forceinline__ void merge_sorted(float *s)
{
    auto exchange = [&](int i, int j) {
        const float a = fminf(s[i], s[j]), b = fmaxf(s[i], s[j]);
        s[i] = a;
        s[j] = b;
    };
#pragma unroll
    for (int i = 0; i < N; ++i)
        exchange(i, i + N);
#pragma unroll
    for (int j = N / 2; j > 0; j >>= 1)
#pragma unroll
        for (int i = j; i + j < 2 * N; i += 2 * j)
#pragma unroll
            for (int q = 0; q < j; ++q)
                exchange(i + q, i + q + j);
}

// A lower bound of sum_j min_p (x_j - s_p)^2 for coefficients c: the chord
// table's value (see the top of the file) less a bound on its rounding.
//
// With u = 2^-24, A = max |s_p|, W = s_n - s_0, X = max |x| and Z = X + A, the
// binary32 roundings move the result by at most u times
//   the subset sums (three additions)                       768 A Z
//   midpoints (256 W A), gaps s_p - s_(p-1) (256 W Z)
//   the cell: 2 m and the values are placed to within 12 u X, and slopes
//     differ by at most 128 (a neighbour's chord, a value counted one cell
//     off)                                                  2 x 1536 W X
//   the chord's slope, value at 0 and result                1024 W Z
//   four running sums of the gaps' products, their total    1536 W Z + 768 Z^2
//   the sum about s_n and the difference                    640 Z^2 + 256 W Z
// which is less than 2300 Z^2 + 6700 W Z.
template <int K>
__device__ __forceinline__ float entry_bound(const EncodeLds &L, const GroupStats &t, const uint16_t *c)
{
    constexpr int NS = 1 << K;
    float s[NS];
    s[0] = 0.0f;
    auto add_plane = [&](auto n_, uint16_t ci) {
        constexpr int N = decltype(n_)::value;
        const float f = half_bits_to_float(ci);
#pragma unroll
        for (int i = 0; i < N; ++i)
            s[N + i] = s[i] + f;
        merge_sorted<N>(s);
    };
    add_plane(std::integral_constant<int, 1>{}, c[0]);
    if constexpr (K > 1)
        add_plane(std::integral_constant<int, 2>{}, c[1]);
    if constexpr (K > 2)
        add_plane(std::integral_constant<int, 4>{}, c[2]);
    if constexpr (K > 3)
        add_plane(std::integral_constant<int, 8>{}, c[3]);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 1; p < NS; ++p) {
        const float m2 = s[p] + s[p - 1], gap = s[p] - s[p - 1];
        const float2 ch = L.cell[cell_of(t, m2)];
        acc[p & 3] = fmaf(gap, fmaf(ch.y, m2, ch.x), acc[p & 3]);
    }
    const float sn = s[NS - 1], W = sn - s[0];
    const float Z = t.X + fmaxf(fabsf(s[0]), fabsf(sn));
    const float about = fmaf((float)GROUP * sn, sn, fmaf(-sn, t.T2, t.S2));
    const float tol = 0x1p-24f * Z * fmaf(2300.f, Z, 6700.f * W);
    return t.X > ENC_SCREEN_MAX ? -3e38f : about - ((acc[0] + acc[1]) + (acc[2] + acc[3])) - tol;
}

// Scores the lanes' coefficient sets c (`want`: the lane has one, `v`: its
// lower bound) on the group.  Every set whose error may be the smallest of
// them, or equal to it, and at most `ub` gets its MSE by the definition's
// order; the others (and lanes without a set) return infinity.  ub: an upper
// bound on the error sum of interest, lowered to the smallest one found.
template <int K>
__device__ double score_lanes(EncodeLds &L, const uint16_t *c, bool want, float v, double d0, double d1, double &ub)
{
    const int lane = threadIdx.x;
    double mse = __builtin_inf();
    uint64_t left = __ballot(want && !(v > f32_above(ub)));
    uint32_t w[(K + 1) / 2];
#pragma unroll
    for (int i = 0; i < (K + 1) / 2; ++i)
        w[i] = (uint32_t)c[2 * i] | (2 * i + 1 < K ? (uint32_t)c[2 * i + 1] << 16 : 0u);
    // the terms of the lane's two elements for the set of lane q
    auto terms = [&](int q, double &e0, double &e1) {
        uint16_t cq[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t wq = (uint32_t)__builtin_amdgcn_readlane((int)w[i / 2], q);
            cq[i] = (uint16_t)(i & 1 ? wq >> 16 : wq & 0xffffu);
        }
        double sums[1 << K];
        subset_sums<K>(cq, sums);
        e0 = nearest_sq<K>(sums, d0);
        e1 = nearest_sq<K>(sums, d1);
    };
    double tsum = __builtin_inf();
    bool first = true, many = false;
    while (left) {
        int q = __ffsll((unsigned long long)left) - 1;
        if (first) {  // the lowest bound first: its error drops most of the others
            const float vm = wave_min_f32((left >> lane) & 1 ? v : __builtin_inff());
            const uint64_t at = __ballot(((left >> lane) & 1) && v == vm);
            q = at ? __ffsll((unsigned long long)at) - 1 : q;
        }
        double e0, e1;
        terms(q, e0, e1);
        const double s = wave_sum_f64(e0 + e1);
        if (lane == q)
            tsum = s;
        ub = fmin(ub, s * (1.0 + ENC_ORDER_EPS));
        left &= __ballot(!(v > f32_above(ub)));
        many = first && __popcll(left) > enc_serial(K);  // (the set just scored among them)
        if (many)
            break;
        left &= ~(1ull << q);
        first = false;
    }
    if (many) {  // a lane per set, the elements in order
        if ((left >> lane) & 1) {
            double sums[1 << K];
            subset_sums<K>(c, sums);
            mse = entry_mse<K>(L.D, sums);
        }
        return mse;
    }
    left = __ballot(tsum * (1.0 - ENC_ORDER_EPS) <= ub && tsum < __builtin_inf());
    while (left) {
        const int q = __ffsll((unsigned long long)left) - 1;
        left &= left - 1;
        double e0, e1;
        terms(q, e0, e1);
        __syncthreads();  // the last reads of E are done
        L.E[lane] = e0;
        L.E[lane + 64] = e1;
        __syncthreads();
        double err = 0.0;
#pragma unroll 16
        for (int j = 0; j < GROUP; ++j)
            err += L.E[j];
        if (lane == q)
            mse = err / (double)GROUP;
    }
    return mse;
}

template <int K>
struct GroupChoice {
    uint16_t c[K];
    double mse;
    int entry;  // index in the grid, -1 for the no-admissible-entry fallback
};

__device__ __forceinline__ int wave_min_int(int v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        v = min(v, __shfl_xor(v, off));
    return v;
}

// Algorithm 1 over the group in L.D (d0, d1: the lane's elements lane and
// lane + 64; st and L.cell: group_table's).  Every lane returns the same choice.
template <int K, bool SCREENED>
__device__ GroupChoice<K> search_group(const EncodeArgs &a, EncodeLds &L, const GroupStats &st, double d0, double d1)
{
    const int lane = threadIdx.x;
    double sum = 0.0;  // in element order
#pragma unroll 16
    for (int j = 0; j < GROUP; ++j)
        sum += L.D[j];
    const double avg = sum / (double)GROUP;

    const double s_max = 1.1 * (st.mx - st.mn);
    const double s_min = 2.0 * st.q95;
    const double s_gran = (s_max - s_min) / (double)a.n_scale;
    const double b_max = 2.0 * fabs(avg) / (double)K;
    const double b_min = -b_max;
    const double b_gran = (b_max - b_min) / (double)a.n_bias;
    const double r1_gran = 0.5 / (double)a.n_ratio1;
    const double r2_gran = 1.0 / (double)a.n_ratio2;
    const int per_r = a.n_scale * a.n_bias;
    const int n_entries = (a.n_ratio1 + a.n_ratio2) * per_r;

    auto ratio_of = [&](int ir) {
        return ir < a.n_ratio1 ? -1.0 + (double)(ir + 1) * r1_gran : -2.0 + (double)(ir - a.n_ratio1) * r2_gran;
    };
    auto scale_of = [&](int js) { return s_min + (double)(js + 1) * s_gran; };
    auto bias_of = [&](int kb) { return b_min + (double)kb * b_gran; };
    // an entry's coefficients; false if it is not admissible
    auto entry_at = [&](int e, uint16_t *c) {
        const double s = scale_of((e / a.n_bias) % a.n_scale);
        EntryShape<K> sh;
        sh.set(ratio_of(e / per_r), s, a.normalise != 0);
        return s > 0.0 && sh.coeffs(bias_of(e % a.n_bias), c);
    };

    double best_mse = __builtin_inf(), ub = __builtin_inf();  // ub: on the smallest error sum
    int best_e = -1;
    if constexpr (!SCREENED) {  // a lane per entry, the elements in order
        double mse = __builtin_inf();
        int e = -1;
        for (int e0 = 0; e0 < n_entries; e0 += ENC_THREADS) {
            uint16_t c[K];
            const int ei = e0 + lane;
            double m = __builtin_inf();
            if (ei < n_entries && entry_at(ei, c)) {
                double sums[1 << K];
                subset_sums<K>(c, sums);
                m = entry_mse<K>(L.D, sums);
            }
            if (m < mse) {
                mse = m;
                e = ei;
            }
        }
        best_mse = wave_min_f64(mse);
        if (best_mse < __builtin_inf())
            best_e = wave_min_int(mse == best_mse ? e : INT_MAX);
    }
    for (int e0 = 0; SCREENED && e0 < n_entries; e0 += ENC_CHUNK) {
        const int left = n_entries - e0;
        const int run = min(ENC_RUN, (left + ENC_THREADS - 1) / ENC_THREADS);
        // Calls f(i, entry, its coefficients or null where it is not admissible)
        // for the lane's run of entries.
        auto walk = [&](auto f) {
            const int e1 = e0 + lane * run;
            int ir = e1 / per_r, js = (e1 / a.n_bias) % a.n_scale, kb = e1 % a.n_bias;
            double s = 0.0;
            EntryShape<K> sh;
            for (int i = 0; i < run; ++i) {
                uint16_t c[K];
                bool ok = false;
                if (e1 + i < n_entries) {
                    if (i == 0 || kb == 0) {
                        s = scale_of(js);
                        sh.set(ratio_of(ir), s, a.normalise != 0);
                    }
                    ok = s > 0.0 && sh.coeffs(bias_of(kb), c);
                    if (++kb == a.n_bias) {
                        kb = 0;
                        if (++js == a.n_scale) {
                            js = 0;
                            ++ir;
                        }
                    }
                }
                f(i, e1 + i, ok ? c : (const uint16_t *)nullptr);
            }
        };
        // lower bounds of the lane's run of entries
        float vmin = __builtin_inff();
        int emin = -1;
        walk([&](int i, int e, const uint16_t *c) {
            float v = __builtin_inff();
            if (c) {
                v = entry_bound<K>(L, st, c);
                if (emin < 0 || v < vmin) {
                    vmin = v;
                    emin = e;
                }
            }
            L.lb[i * ENC_THREADS + lane] = v;
        });
        // the entry with the lowest bound, scored: its error drops most others
        const uint64_t have = __ballot(emin >= 0);
        if (have == 0)  // no admissible entry in this chunk
            continue;
        const float vm = wave_min_f32(vmin);
        const uint64_t at = __ballot(emin >= 0 && vmin == vm);
        const int es = __builtin_amdgcn_readlane(emin, __ffsll((unsigned long long)(at ? at : have)) - 1);
        {
            uint16_t c[K];
            entry_at(es, c);
            double sums[1 << K];
            subset_sums<K>(c, sums);
            ub = fmin(ub, wave_sum_f64(nearest_sq<K>(sums, d0) + nearest_sq<K>(sums, d1)) * (1.0 + ENC_ORDER_EPS));
        }
        // entries that may win or tie (an inadmissible one has v = infinity)
        auto kept = [&](int i) {
            const float v = L.lb[i * ENC_THREADS + lane];
            return !(v > f32_above(ub)) && v < __builtin_inff();
        };
        int n = 0;
        for (int i = 0; i < run; ++i) {
            const bool k = kept(i);
            const uint64_t m = __ballot(k);
            const int slot = n + __popcll(m & ((1ull << lane) - 1));
            if (k && slot < ENC_LIST)
                L.list[slot] = e0 + lane * run + i;
            n += __popcll(m);
        }
        __syncthreads();
        double mse = __builtin_inf();
        int e = -1;
        if (n <= ENC_LIST) {
            uint16_t c[K] = {};
            float v = __builtin_inff();
            if (lane < n) {
                e = L.list[lane];
                entry_at(e, c);
                v = L.lb[(e - e0) % run * ENC_THREADS + (e - e0) / run];
            }
            mse = score_lanes<K>(L, c, lane < n, v, d0, d1, ub);
        } else {  // a lane per entry, the elements in order
            walk([&](int i, int ei, const uint16_t *c) {
                double m = __builtin_inf();
                if (c && kept(i)) {
                    double sums[1 << K];
                    subset_sums<K>(c, sums);
                    double err = 0.0;
                    for (int j0 = 0; j0 < GROUP && err <= ub; j0 += 16)
#pragma unroll(K <= 2 ? 16 : 4)
                        for (int j = j0; j < j0 + 16; ++j)
                            err += nearest_sq<K>(sums, L.D[j]);
                    if (err <= ub)  // (else it can neither win nor tie)
                        m = err / (double)GROUP;
                }
                if (m < mse) {
                    mse = m;
                    e = ei;
                }
                ub = fmin(ub, wave_min_f64(m) * (double)GROUP);
            });
        }
        // smallest error, lowest entry index among equal errors
        const double m = wave_min_f64(mse);
        if (m < best_mse) {  // (an equal one of an earlier chunk comes first)
            best_mse = m;
            best_e = wave_min_int(mse == m ? e : INT_MAX);
        }
        __syncthreads();  // lb and list are read before the next chunk's
    }

    GroupChoice<K> out;
    if (best_e >= 0) {
        entry_at(best_e, out.c);
    } else {  // no admissible entry
        out.c[0] = f64_to_f16_rne(avg);
#pragma unroll
        for (int i = 1; i < K; ++i)
            out.c[i] = 0;
        double sums[1 << K];
        subset_sums<K>(out.c, sums);
        best_mse = entry_mse<K>(L.D, sums);
    }
    out.mse = best_mse;
    out.entry = best_e;
    return out;
}

// The bitvector assignment for coefficient set c (each of the lane's two
// elements takes the pattern of its nearest subset sum) and the group's
// stores: plane i by lane i, the coefficients, the MSE by lane 0.
template <int K>
__device__ __forceinline__ void store_group(const EncodeArgs &a, size_t grp, const uint16_t *c, double d0,
                                            double d1, double mse)
{
    const int lane = threadIdx.x;
    double sums[1 << K];
    subset_sums<K>(c, sums);
    double dd;
    const int p0 = nearest<K>(sums, d0, dd), p1 = nearest<K>(sums, d1, dd);
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const uint64_t m0 = __ballot((p0 >> i) & 1), m1 = __ballot((p1 >> i) & 1);
        if (lane == i) {
            uint32_t *pl = a.planes + (grp * K + i) * 4;
            *(uint4 *)pl = make_uint4((uint32_t)m0, (uint32_t)(m0 >> 32), (uint32_t)m1, (uint32_t)(m1 >> 32));
            a.coeffs[grp * K + i] = c[i];
        }
    }
    if (lane == 0 && a.mse)
        a.mse[grp] = mse;
}

template <int K, bool SCREENED>
__global__ void __launch_bounds__(ENC_THREADS) encode_kernel(EncodeArgs a)
{
    __shared__ EncodeLds L;
    const int lane = threadIdx.x;
    const int G = a.I / GROUP;
    const size_t grp = blockIdx.x;
    const size_t o = grp / G, g = grp % G;
    const float *src = a.W + o * (size_t)a.I + g * GROUP;

    const float x0 = src[lane], x1 = src[lane + 64];
    const double d0 = (double)x0, d1 = (double)x1;
    L.D[lane] = d0;
    L.D[lane + 64] = d1;
    const GroupStats st = group_table<SCREENED>(L, x0, x1);
    const GroupChoice<K> r = search_group<K, SCREENED>(a, L, st, d0, d1);
    store_group<K>(a, grp, r.c, d0, d1, r.mse);
}

// The encoder with the cache of Sec. 4.2 (last paragraph and its footnote):
// one wavefront per row, its groups in index order.  Lane s holds cache slot
// s (a coefficient set the full search chose for one of the row's last
// `slots` searched groups, and that group's insertion number; the oldest set
// is replaced first).  For each group every held set is scored with the
// search's MSE (screened like the entries of a search); the smallest --
// the oldest among equal ones -- is taken if it is strictly below the mean
// MSE of the row's earlier groups (binary64 sum in group order over their
// count), otherwise the full search runs and its choice enters the cache
// (the no-admissible-entry fallback does not).  The first group of a row
// always searches; with slots = 0 the result is the plain encoder's.
template <int K, bool SCREENED>
__global__ void __launch_bounds__(ENC_THREADS) encode_cached_kernel(EncodeArgs a, int slots, uint8_t *hits)
{
    __shared__ EncodeLds L;
    const int lane = threadIdx.x;
    const int G = a.I / GROUP;
    const size_t o = blockIdx.x;
    uint16_t cs[K];  // this lane's cached set
#pragma unroll
    for (int i = 0; i < K; ++i)
        cs[i] = 0;
    int seq = INT_MAX;             // its insertion number
    int n_cached = 0, n_ins = 0;   // wavefront-uniform
    double mse_sum = 0.0;          // wavefront-uniform
    for (int g = 0; g < G; ++g) {
        const size_t grp = o * G + g;
        const float *src = a.W + o * (size_t)a.I + (size_t)g * GROUP;
        const float x0 = src[lane], x1 = src[lane + 64];
        const double d0 = (double)x0, d1 = (double)x1;
        __syncthreads();  // the previous group's reads of L are done
        L.D[lane] = d0;
        L.D[lane + 64] = d1;
        const GroupStats st = group_table<SCREENED>(L, x0, x1);
        bool hit = false;
        uint16_t c[K];
        double mse = 0.0;
        if (g > 0 && n_cached > 0) {
            const double avg = mse_sum / (double)g;
            // a set whose lower bound is above the mean cannot be taken
            const bool held = lane < n_cached;
            const float v = held ? (SCREENED ? entry_bound<K>(L, st, cs) : -3e38f) : __builtin_inff();
            double ub = avg * (double)GROUP;
            const double m = score_lanes<K>(L, cs, held, v, d0, d1, ub);
            const double best = wave_min_f64(m);
            if (best < avg) {  // wavefront-uniform
                const int oldest = wave_min_int(lane < n_cached && m == best ? seq : INT_MAX);
                const int wl = __ffsll((unsigned long long)__ballot(lane < n_cached && seq == oldest)) - 1;
#pragma unroll
                for (int i = 0; i < K; ++i)
                    c[i] = (uint16_t)__shfl((int)cs[i], wl);
                mse = best;
                hit = true;
            }
        }
        if (!hit) {
            const GroupChoice<K> r = search_group<K, SCREENED>(a, L, st, d0, d1);
#pragma unroll
            for (int i = 0; i < K; ++i)
                c[i] = r.c[i];
            mse = r.mse;
            if (r.entry >= 0 && slots > 0) {
                if (lane == n_ins % slots) {
#pragma unroll
                    for (int i = 0; i < K; ++i)
                        cs[i] = c[i];
                    seq = n_ins;
                }
                ++n_ins;
                n_cached = min(n_cached + 1, slots);
            }
        }
        store_group<K>(a, grp, c, d0, d1, mse);
        if (lane == 0 && hits)
            hits[grp] = hit ? 1 : 0;
        mse_sum += mse;
    }
}

// The kernel (KERNEL<K, SCREENED>) for k planes and the grid of a.
#define SBVR_ENCODE_KERNEL(KERNEL, k, screened)                                                                \
    ((screened) ? ((k) == 4   ? (const void *)KERNEL<4, true>                                                  \
                   : (k) == 3 ? (const void *)KERNEL<3, true>                                                  \
                   : (k) == 2 ? (const void *)KERNEL<2, true>                                                  \
                              : (const void *)KERNEL<1, true>)                                                 \
                : ((k) == 4   ? (const void *)KERNEL<4, false>                                                 \
                   : (k) == 3 ? (const void *)KERNEL<3, false>                                                 \
                   : (k) == 2 ? (const void *)KERNEL<2, false>                                                 \
                              : (const void *)KERNEL<1, false>))

static bool screened(const EncodeArgs &a, int k)
{
    return ((a.n_ratio1 + a.n_ratio2) * a.n_scale * a.n_bias) << k > ENC_PLAIN_SUMS;
}

int launch_encode(int O, int I, int k, const float *W, int n_ratio1, int n_ratio2, int n_scale, int n_bias,
                  int normalise, uint32_t *planes, uint16_t *coeffs, double *mse, hipStream_t stream)
{
    EncodeArgs a = {W, planes, coeffs, mse, O, I, n_ratio1, n_ratio2, n_scale, n_bias, normalise};
    const size_t groups = (size_t)O * (I / GROUP);
    const void *fn = SBVR_ENCODE_KERNEL(encode_kernel, k, screened(a, k));
    void *args[] = {&a};
    return launch_kernel(fn, dim3((unsigned)groups), dim3(ENC_THREADS), 0, stream, args);
}

int launch_encode_cached(int O, int I, int k, const float *W, int n_ratio1, int n_ratio2, int n_scale, int n_bias,
                         int normalise, int slots, uint32_t *planes, uint16_t *coeffs, double *mse, uint8_t *hits,
                         hipStream_t stream)
{
    EncodeArgs a = {W, planes, coeffs, mse, O, I, n_ratio1, n_ratio2, n_scale, n_bias, normalise};
    const void *fn = SBVR_ENCODE_KERNEL(encode_cached_kernel, k, screened(a, k));
    void *args[] = {&a, &slots, &hits};
    return launch_kernel(fn, dim3((unsigned)O), dim3(ENC_THREADS), 0, stream, args);
}

}  // namespace sbvr
