// Decoding SBVR weights in registers (the prefill paths).
//
// A weight is one of the 2^k subset sums of its group's coefficients (Sec.
// 4.1), rounded once to binary16.  A lane that decodes weights of one row
// holds the row's 2^k sums as bytes, low and high ones apart, in up to eight
// registers; byte permutes then look up four weights at a time.  Against a
// table in LDS, one read per weight, this trades about 2 vector instructions
// per weight for the LDS reads, whose bank conflicts (random entries, about 6
// LDS cycles per 64 lookups, shared by a CU's four SIMDs) bounded the prefill
// kernels.
#pragma once

#include "device_ops.h"
#include "f16_round.h"

namespace sbvr {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// A row's subset sums: byte j of lo[i] / hi[i] belongs to subset 4 i + j.
template <int K>
struct RowTable {
    static constexpr int N = K < 2 ? 1 : (1 << K) / 4;
    uint32_t lo[N], hi[N];
};

// The k coefficients of a row and group, packed pairs of binary16.
template <int K>
struct RowCoefs {
    uint32_t w[(K + 1) / 2];
};

// True when binary32 subset sums of these coefficients are exact: the
// condition of f16_sums_exact_in_f32 (exponents spanning at most 11) on packed
// 16-bit operations; a set at the limit may be refused, none is wrongly taken
// (a magnitude's pattern less one has an exponent no larger than its own, and
// turns zero into the largest value).
template <int K>
__device__ __forceinline__ bool row_sums_exact_in_f32(const RowCoefs<K> &c)
{
    typedef unsigned short u2_t __attribute__((ext_vector_type(2)));
    const u2_t one = {1, 1};
    u2_t mx = __builtin_bit_cast(u2_t, c.w[0] & 0x7fff7fffu), mn = mx - one;
    if constexpr (K > 2) {
        const u2_t v = __builtin_bit_cast(u2_t, c.w[1] & 0x7fff7fffu);
        mx = __builtin_elementwise_max(mx, v);
        mn = __builtin_elementwise_min(mn, v - one);
    }
    const int hi = max((int)mx[0], (int)mx[1]), lo = min((int)mn[0], (int)mn[1]);
    return (hi >> 10) - (lo >> 10) <= 11;
}

__device__ __forceinline__ uint32_t pack_f16_rne(float a, float b)
{
    typedef float f2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2_t{a, b}, h2_t));
}

// The table from its entries (binary16, pairs): for k >= 3 the lanes l and
// l + 32 hold the same row, each has the half of the subsets whose top bit is
// its half, and the halves trade.
template <int K>
struct RowEntries {
    static constexpr int PER = K >= 3 ? (1 << K) / 2 : (1 << K);  // subsets per lane
    static constexpr int LOW = K >= 3 ? K - 1 : K;                // planes the lane's subsets vary
    uint32_t e[PER / 2];
};

template <int K>
__device__ __forceinline__ RowTable<K> row_table(const RowEntries<K> &r)
{
    const uint32_t *e = r.e;
    RowTable<K> t;
    if constexpr (K == 1) {
        t.lo[0] = __builtin_amdgcn_perm(e[0], e[0], 0x02000200u);
        t.hi[0] = __builtin_amdgcn_perm(e[0], e[0], 0x03010301u);
    } else if constexpr (K == 2) {
        t.lo[0] = __builtin_amdgcn_perm(e[1], e[0], 0x06040200u);
        t.hi[0] = __builtin_amdgcn_perm(e[1], e[0], 0x07050301u);
    } else {
        constexpr int H = RowEntries<K>::PER / 4;  // registers of a half
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const uint32_t l = __builtin_amdgcn_perm(e[2 * i + 1], e[2 * i], 0x06040200u);
            const uint32_t h = __builtin_amdgcn_perm(e[2 * i + 1], e[2 * i], 0x07050301u);
            const auto sl = __builtin_amdgcn_permlane32_swap(l, l, false, false);
            const auto sh = __builtin_amdgcn_permlane32_swap(h, h, false, false);
            t.lo[i] = sl[0];
            t.lo[H + i] = sl[1];
            t.hi[i] = sh[0];
            t.hi[H + i] = sh[1];
        }
    }
    return t;
}

template <int K>
__device__ __forceinline__ uint32_t row_coef(const RowCoefs<K> &c, int i)
{
    return i & 1 ? c.w[i / 2] >> 16 : c.w[i / 2] & 0xffffu;
}

// The table of a row whose group has coefficients c, by binary32 sums (exact,
// whatever their order, where row_sums_exact_in_f32), rounded once.
template <int K>
__device__ __forceinline__ RowTable<K> row_table32(const RowCoefs<K> &c, int half)
{
    constexpr int PER = RowEntries<K>::PER, LOW = RowEntries<K>::LOW;
    float s[PER];
    s[0] = 0.f;
    if constexpr (K >= 3)
        s[0] = half ? half_bits_to_float(row_coef<K>(c, K - 1)) : 0.f;
#pragma unroll
    for (int i = 0; i < LOW; ++i) {
        const float f = half_bits_to_float(row_coef<K>(c, i));
#pragma unroll
        for (int p = 0; p < (1 << i); ++p)
            s[(1 << i) + p] = s[p] + f;
    }
    RowEntries<K> r;
#pragma unroll
    for (int q = 0; q < PER / 2; ++q)
        r.e[q] = pack_f16_rne(s[2 * q], s[2 * q + 1]);
    return row_table<K>(r);
}

// The same by binary64 sums: exact for at most four binary16 terms.
template <int K>
__device__ __forceinline__ RowTable<K> row_table64(const RowCoefs<K> &c, int half)
{
    constexpr int PER = RowEntries<K>::PER, LOW = RowEntries<K>::LOW;
    RowEntries<K> r;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int sub = K >= 3 ? p + (half << LOW) : p;
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < K; ++i)
            s += ((sub >> i) & 1) ? (double)half_bits_to_float(row_coef<K>(c, i)) : 0.0;
        const uint32_t h = f64_to_f16_odd(s);
        r.e[p / 2] = p & 1 ? r.e[p / 2] | (h << 16) : h;
    }
    return row_table<K>(r);
}

// The same tables where four lanes (l, l + 16, l + 32, l + 48) hold a row: for
// k = 4 each sums a quarter of the subsets (the ones whose top two bits are its
// quarter), for k = 3 a half; then they trade.
template <int K>
struct QuarterEntries {
    static constexpr int LOW = K >= 2 ? 2 : 1;  // planes the lane's subsets vary
    static constexpr int PER = 1 << LOW;
    uint32_t e[PER / 2];
};

template <int K>
__device__ __forceinline__ RowTable<K> quarter_table(const QuarterEntries<K> &r)
{
    const uint32_t *e = r.e;
    RowTable<K> t;
    if constexpr (K == 1) {
        t.lo[0] = __builtin_amdgcn_perm(e[0], e[0], 0x02000200u);
        t.hi[0] = __builtin_amdgcn_perm(e[0], e[0], 0x03010301u);
    } else {
        const uint32_t l = __builtin_amdgcn_perm(e[1], e[0], 0x06040200u);
        const uint32_t h = __builtin_amdgcn_perm(e[1], e[0], 0x07050301u);
        if constexpr (K == 2) {
            t.lo[0] = l;
            t.hi[0] = h;
        } else {
            auto trade = [](uint32_t v, uint32_t *out) {
                if constexpr (K == 4) {
                    const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
                    const auto a = __builtin_amdgcn_permlane16_swap(s[0], s[0], false, false);
                    const auto b = __builtin_amdgcn_permlane16_swap(s[1], s[1], false, false);
                    out[0] = a[0];
                    out[1] = a[1];
                    out[2] = b[0];
                    out[3] = b[1];
                } else {
                    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
                    out[0] = a[0];
                    out[1] = a[1];
                }
            };
            trade(l, t.lo);
            trade(h, t.hi);
        }
    }
    return t;
}

template <int K>
__device__ __forceinline__ RowTable<K> quarter_table32(const RowCoefs<K> &c, int quarter)
{
    constexpr int PER = QuarterEntries<K>::PER, LOW = QuarterEntries<K>::LOW;
    float s[PER];
    s[0] = 0.f;
#pragma unroll
    for (int i = LOW; i < K; ++i)
        s[0] += (quarter >> (i - LOW)) & 1 ? half_bits_to_float(row_coef<K>(c, i)) : 0.f;
#pragma unroll
    for (int i = 0; i < LOW; ++i) {
        const float f = half_bits_to_float(row_coef<K>(c, i));
#pragma unroll
        for (int p = 0; p < (1 << i); ++p)
            s[(1 << i) + p] = s[p] + f;
    }
    QuarterEntries<K> r;
#pragma unroll
    for (int q = 0; q < PER / 2; ++q)
        r.e[q] = pack_f16_rne(s[2 * q], s[2 * q + 1]);
    return quarter_table<K>(r);
}

template <int K>
__device__ __forceinline__ RowTable<K> quarter_table64(const RowCoefs<K> &c, int quarter)
{
    constexpr int PER = QuarterEntries<K>::PER, LOW = QuarterEntries<K>::LOW;
    QuarterEntries<K> r;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int sub = p + (quarter << LOW);
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < K; ++i)
            s += ((sub >> i) & 1) ? (double)half_bits_to_float(row_coef<K>(c, i)) : 0.0;
        const uint32_t h = f64_to_f16_odd(s);
        r.e[p / 2] = p & 1 ? r.e[p / 2] | (h << 16) : h;
    }
    return quarter_table<K>(r);
}

// Boolean functions of three registers.  v_bitop3_b32 issues in about 2.6
// cycles with two or more wavefronts on a SIMD, v_bfi_b32 and v_and_or_b32 in
// about 4.6; an operand in a scalar register costs the same 4.3, so the masks
// are kept in vector registers.
__device__ __forceinline__ uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b)  // m ? a : b
{
    return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA);
}

__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t m, uint32_t c)  // (a & m) | c
{
    return __builtin_amdgcn_bitop3_b32(a, m, c, 0xEA);
}

// Masks of the decoding, in vector registers.
struct DecodeMasks {
    uint32_t m33, m55, mff, m04, id;

    __device__ __forceinline__ void set()
    {
        asm("v_mov_b32 %0, 0x33333333" : "=v"(m33));
        asm("v_mov_b32 %0, 0x55555555" : "=v"(m55));
        asm("v_mov_b32 %0, 0x00ff00ff" : "=v"(mff));
        asm("v_mov_b32 %0, 0x04040404" : "=v"(m04));
        asm("v_mov_b32 %0, 0x03020100" : "=v"(id));
    }
};

// The subset indices of 32 elements, eight per register: element 8v+p of a
// device plane word sits at bit 4p+v, so nibble p of plane word w_i holds bits
// v of elements 8v+p; transposing the 4 x 4 (plane, v) bits of every nibble
// gives pat[v], whose nibble p is the index of element 8v+p.
template <int K>
__device__ __forceinline__ void subset_indices(const DecodeMasks &m, const uint32_t *w, uint32_t *pat)
{
    if constexpr (K == 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            pat[v] = (w[0] >> v) & 0x11111111u;
    } else {
        const uint32_t w0 = w[0], w1 = w[1], w2 = K > 2 ? w[K > 2 ? 2 : 0] : 0u, w3 = K > 3 ? w[K > 3 ? 3 : 0] : 0u;
        const uint32_t a0 = bit_select(m.m33, w0, w2 << 2), a2 = bit_select(m.m33, w0 >> 2, w2);
        const uint32_t a1 = bit_select(m.m33, w1, w3 << 2), a3 = bit_select(m.m33, w1 >> 2, w3);
        pat[0] = bit_select(m.m55, a0, a1 << 1);
        pat[1] = bit_select(m.m55, a0 >> 1, a1);
        pat[2] = bit_select(m.m55, a2, a3 << 1);
        pat[3] = bit_select(m.m55, a2 >> 1, a3);
    }
}

// Four lookups: byte j of the result is the byte of the entry whose index is
// byte j of `ix` (its low three bits), among the upper eight entries where byte
// j of `up` is 4 + j instead of j.
template <int K>
__device__ __forceinline__ uint32_t lookup4(const uint32_t *t, uint32_t ix, uint32_t up)
{
    if constexpr (K <= 2) {
        return __builtin_amdgcn_perm(t[0], t[0], ix);
    } else if constexpr (K == 3) {
        return __builtin_amdgcn_perm(t[1], t[0], ix);
    } else {
        return __builtin_amdgcn_perm(__builtin_amdgcn_perm(t[3], t[2], ix), __builtin_amdgcn_perm(t[1], t[0], ix), up);
    }
}

// The eight binary16 weights of `pat`, in element order.
template <int K>
__device__ __forceinline__ uint4 decode8(const DecodeMasks &m, const RowTable<K> &t, uint32_t pat)
{
    constexpr uint32_t IX = K == 4 ? 0x07070707u : 0x0f0f0f0fu;
    // low nibbles of the bytes: elements 0, 1, 4, 5 and 2, 3, 6, 7
    const uint32_t a = bit_select(m.mff, pat, pat << 4), b = bit_select(m.mff, pat >> 8, pat >> 4);
    const uint32_t ua = and_or(a >> 1, m.m04, m.id), ub = and_or(b >> 1, m.m04, m.id);
    const uint32_t la = lookup4<K>(t.lo, a & IX, ua), ha = lookup4<K>(t.hi, a & IX, ua);
    const uint32_t lb = lookup4<K>(t.lo, b & IX, ub), hb = lookup4<K>(t.hi, b & IX, ub);
    return make_uint4(__builtin_amdgcn_perm(ha, la, 0x05010400u), __builtin_amdgcn_perm(hb, lb, 0x05010400u),
                      __builtin_amdgcn_perm(ha, la, 0x07030602u), __builtin_amdgcn_perm(hb, lb, 0x07030602u));
}

}  // namespace sbvr
