// Prefill GEMM on SBVR weights: Y[t][o] = sum_j X[t][j] * fp16(w_hat[o][j])
// for a prompt of T tokens (the paper's prefill design decompresses the
// weights to binary16 and multiplies them on the tensor cores, Sec. 5.1; here
// the binary16 matrix never goes to memory).
//
// The decoded weight fp16(w_hat) is the correctly rounded subset sum of its
// group's coefficients (Sec. 4.1), the same value sbvr_decompress writes, so
// the result equals X times the decompressed matrix with fp32 accumulation.
//
// Two kernels, both decoding in registers (row_decode.h): a lane holds the
// subset-sum table of one weight row and the subset indices of its elements of
// a group, looks up eight weights per step with byte permutes and feeds them
// to the matrix cores as the B operand; the activations, staged in LDS by
// direct loads, are the A operand.  The groups of the inner dimension are
// split into K-slices over wavefronts, whose partial sums are added through
// LDS in a fixed order.
//
//   * prefill_kernel: v_mfma_f32_32x32x16_f16.  A wavefront owns RT column
//     tiles of 32 weight rows, TT token tiles of 32 and one K-slice; a
//     workgroup of eight holds R row groups times S = 8 / R K-slices, the R
//     wavefronts of a K-slice sharing its activations.
//   * prefill_short_kernel: v_mfma_f32_16x16x32_f16.  A workgroup owns one
//     tile of 16 weight rows and TT token tiles of 16, a wavefront per K-slice:
//     twice the workgroups per matrix and half the decoding per wavefront and
//     group, for prompts up to about 32 tokens and small matrices.
//
// What bounds them: vector instruction issue.  A wavefront decodes 32 rows x
// 128 weights with about 350 instructions (k = 4; 132 byte permutes at 4.5
// cycles each, most of the others at 2.6-4), beside 8 matrix-core instructions
// per 32 tokens; at 512 tokens the two are about equal and the clock (1.75-1.9
// GHz under this load) sets the time.  The earlier kernels looked every weight
// up in an LDS table: random 2-byte reads at 6 LDS cycles per 64 lanes and CU
// or more, which the four SIMDs of a CU share.  Llama-3-8B shapes, k = 4, back
// to back over rotating weights, before -> after (us):
//   tokens            1            37           128          512
//   4096 x 4096     10.9 -> 6.7  17.5 -> 10.3  26.7 -> 13.8  53.6 -> 29.9
//   1024 x 4096     10.3 -> 5.9  11.0 -> 7.0   14.9 -> 10.2  26.7 -> 16.8
//   14336 x 4096    29.1 -> 15.4 50.0 -> 19.1  52.2 -> 30.0  120 -> 75
//   4096 x 14336    27.3 -> 14.9 47.3 -> 25.0  80.0 -> 36.6  166 -> 92
#include "launch.h"
#include "row_decode.h"

#include <math.h>

namespace sbvr {

constexpr size_t PF_LDS_MAX = 160 * 1024;  // LDS of one workgroup on gfx950
constexpr int PF_WAVES = 8;                // wavefronts of a prefill_kernel workgroup
constexpr int PF_CUS = 256;

struct PrefillArgs {
    const uint32_t *planes;  // device plane blocks
    const uint16_t *coeffs;  // device coefficient blocks
    const uint16_t *X;       // binary16 [T][I]
    uint16_t *Y;             // binary16 [T][O]
    int O, I, T, n_tiles, n_gblocks, G, gps;  // gps: groups per K-slice
};

typedef float v16f __attribute__((ext_vector_type(16)));

// One direct load of 1 KiB into LDS: every lane's 16 bytes at `src` to dst +
// 16 lane.  Complete when the wavefront's vector-memory count says so.
__device__ __forceinline__ void load_to_lds(const uint16_t *src, unsigned char *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// Every load the wavefront has issued is complete, the direct ones into LDS
// included (no register waits for those).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

// Orders a wavefront's LDS accesses where no other wavefront shares them.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The k coefficients of a row and group slot b, from the row's place in the
// coefficient block (byte pointer, group slot 0).  k = 3: six bytes at a
// multiple of two, loaded as the two aligned words that hold them and shifted
// into place by row_coefs (not here: that would wait for the load).
template <int K>
__device__ __forceinline__ RowCoefs<K> load_row_coefs(const unsigned char *p, int b)
{
    RowCoefs<K> c;
    p += b * (coefs_per_quad(K) * 2);
    if constexpr (K == 4) {
        const uint2 v = *(const uint2 *)p;
        c.w[0] = v.x;
        c.w[1] = v.y;
    } else if constexpr (K == 3) {
        const uint32_t *v = (const uint32_t *)(p - 2 * (b & 1));
        c.w[0] = v[0];
        c.w[1] = v[1];
    } else if constexpr (K == 2) {
        c.w[0] = *(const uint32_t *)p;
    } else {
        c.w[0] = *(const uint16_t *)p;
    }
    return c;
}

// ... as loaded for group g, zero for a row the device format does not hold.
template <int K>
__device__ __forceinline__ RowCoefs<K> row_coefs(RowCoefs<K> c, int g, bool ok)
{
    if constexpr (K == 3) {
        const int sh = (g & 1) * 16;
        const uint64_t v = (((uint64_t)c.w[1] << 32) | c.w[0]) >> sh;
        c.w[0] = (uint32_t)v;
        c.w[1] = (uint32_t)(v >> 32) & 0xffffu;
    }
#pragma unroll
    for (int i = 0; i < (K + 1) / 2; ++i)
        c.w[i] = ok ? c.w[i] : 0u;
    return c;
}

// ST: activation stages per group (two halve the LDS a stage takes).
template <int K, int RT, int TT, int R, int ST>
__global__ void __launch_bounds__(64 * PF_WAVES) prefill_kernel(PrefillArgs a)
{
    constexpr int S = PF_WAVES / R;
    constexpr int TR = tile_rows(K);
    constexpr int XT = 32 * TT * 256 / ST;  // bytes of a stage's activation tile
    constexpr int SPS = 8 / ST;              // steps per stage
    constexpr unsigned PBLK_B = GB * TR * K * 16, CBLK_B = GB * TR * K * 2;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, w = wave_id();
    const int ks_id = w % S, rg = w / S;  // K-slice and row group of this wavefront
    const int n = lane & 31, kh = lane >> 5;
    unsigned char *xbuf = smem + (size_t)ks_id * 2 * XT;
    const int o_base = (blockIdx.x * R + rg) * 32 * RT, t_base = blockIdx.y * 32 * TT;
    const int g0 = ks_id * a.gps;
    const int rows_dev = a.n_tiles * TR;  // rows held by the device format (padding included)

    v16f acc[RT][TT];
#pragma unroll
    for (int q = 0; q < RT; ++q)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                acc[q][tt][e] = 0.f;

    // The lane's rows (row lane % 32 of each column tile): byte offsets of its
    // plane slots and coefficients in the first gblock's first group.
    unsigned p_lane[RT], c_lane[RT];  // p_lane: of the first slot the lane's half loads (see indices)
    bool row_ok[RT];
#pragma unroll
    for (int q = 0; q < RT; ++q) {
        const int o = min(o_base + 32 * q + n, rows_dev - 1);
        row_ok[q] = o_base + 32 * q + n < rows_dev;
        const unsigned blk = (unsigned)(o / TR) * (unsigned)a.n_gblocks;
        const int r = o % TR;
        constexpr unsigned HALF_B = K >= 3 ? 32 : (K == 2 ? 16 : 0);
        p_lane[q] = blk * PBLK_B + (unsigned)(r * K * 16) + kh * HALF_B;
        c_lane[q] = blk * CBLK_B + (unsigned)coeff_entry(K, r, 0, 0) * 2u;
    }
    const int p_next = K == 3 && kh ? -16 : 16;  // to the second slot
    DecodeMasks masks;
    masks.set();
    struct GroupLoads {
        uint4 p[RT][K >= 3 ? 2 : 1];
        RowCoefs<K> c[RT];
    };
    auto load_group = [&](int g, GroupLoads &L) {
        const unsigned pu = (unsigned)(g / GB) * PBLK_B + (unsigned)(g % GB) * (TR * K * 16);
        const unsigned char *pb = (const unsigned char *)a.planes + pu;
        const unsigned char *cb = (const unsigned char *)a.coeffs + (unsigned)(g / GB) * CBLK_B;
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            L.c[q] = load_row_coefs<K>(cb + c_lane[q], g % GB);
            L.p[q][0] = *(const uint4 *)(pb + p_lane[q]);
            if constexpr (K >= 3)
                L.p[q][1] = *(const uint4 *)(pb + p_lane[q] + p_next);
        }
    };
    // Subset indices of the lane's 64 elements of row tile q: words lane / 32
    // and 2 + lane / 32 of every plane.  The halves of the wavefront load whole
    // slots -- of planes 0, 1 and 2, 3 (k = 4), 0, 1 and 2, 1 (k = 3), 0 and 1
    // (k = 2), 0 both (k = 1) -- and trade words.
    auto indices = [&](const GroupLoads &L, int q, uint32_t *pat) {
        uint32_t w0[4] = {}, w1[4] = {};
        auto trade = [&](uint4 v, int lo, int hi) {  // lo, hi: the planes of the two halves' slots
            const auto x = __builtin_amdgcn_permlane32_swap(v.x, v.y, false, false);
            const auto y = __builtin_amdgcn_permlane32_swap(v.z, v.w, false, false);
            w0[hi] = x[1];
            w1[hi] = y[1];
            w0[lo] = x[0];
            w1[lo] = y[0];
        };
        if constexpr (K >= 3) {
            trade(L.p[q][0], 0, 2);
            trade(L.p[q][1], 1, K == 4 ? 3 : 1);
        } else {
            trade(L.p[q][0], 0, K == 2 ? 1 : 0);
        }
        subset_indices<K>(masks, w0, pat);
        subset_indices<K>(masks, w1, pat + 4);
    };

    // A group's activation tile, loaded straight into LDS by the K-slice's R
    // wavefronts, four tokens (1 KiB) per instruction.  Token t's 256 bytes
    // lie together, its 16-byte chunk c in place c ^ (t % 16), so that the 16
    // tokens of a quarter of an operand read fall on different banks.  Tokens
    // past the prompt read the last one or are left as they are: their results
    // are not stored.
    constexpr int XI = 8 * TT / ST;            // instructions per stage
    constexpr int TPI = 4 * ST, CPT = 16 / ST;  // tokens per instruction, chunks per token
    const int x_rounds = (min(32 * TT, a.T - t_base) + TPI - 1) / TPI;
    auto load_x = [&](int stage, unsigned char *buf) {  // stage: ST per group
#pragma unroll
        for (int q = 0; q < (XI + R - 1) / R; ++q) {
            const int i = rg + q * R;  // wavefront-uniform
            if (i < x_rounds) {
                const int t = TPI * i + lane / CPT;
                const int c = (lane % CPT) ^ (ST == 1 ? t & 15 : (t >> 1) & 7);
                load_to_lds(a.X + (size_t)min(t_base + t, a.T - 1) * a.I + (size_t)stage * (GROUP / ST) + c * 8,
                            buf + i * 1024);
            }
        }
    };
    // the next stage's loads are complete, for all the wavefronts that read it
    auto sync = [&]() {
        wait_loads();
        if constexpr (R == 1)
            wave_sync();
        else
            __syncthreads();
    };

    // The decoding state of a group: tables and subset indices of the row tiles.
    struct GroupState {
        RowTable<K> tab[RT];
        uint32_t pat[RT][8];
    };
    auto prepare = [&](const GroupLoads &L, int g, GroupState &s) {
        bool wide = false;
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            const RowCoefs<K> c = row_coefs<K>(L.c[q], g, row_ok[q]);
            wide = wide || !row_sums_exact_in_f32<K>(c);
            s.tab[q] = row_table32<K>(c, kh);
            indices(L, q, s.pat[q]);
        }
        if (__builtin_amdgcn_ballot_w64(wide) != 0) {  // some row's sums are not exact in binary32
#pragma unroll
            for (int q = 0; q < RT; ++q)
                s.tab[q] = row_table64<K>(row_coefs<K>(L.c[q], g, row_ok[q]), kh);
        }
    };

    const int g_last = min(g0 + a.gps, a.G) - 1, g_first = min(g0, a.G - 1);
    GroupLoads raw;
    load_x(g_first * ST, xbuf);
    load_group(g_first, raw);
    sync();
    // operand reads: token n's chunk of the lane's elements; word lane / 32
    // is chunks 4 (lane / 32) .. of a stage's first 64 elements
    const int x_lane = ST == 1 ? n * 256 + (((n & 15) ^ (4 * kh)) << 4) : n * 128 + ((((n >> 1) & 7) ^ (4 * kh)) << 4);
    auto x_step = [&](int st) { return x_lane ^ (ST == 1 ? ((st & 3) | (st >> 2 << 3)) << 4 : (st & 3) << 4); };
    int buf = 0;
    for (int j = 0; j < a.gps; ++j) {
        const int g = g0 + j;
        // past the K-slice's last group: it is loaded again and not used
        const int gn = max(min(g + 1, g_last), g_first);
        GroupState cur;
        prepare(raw, min(g, a.G - 1), cur);
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            const int next_stage = s + 1 < ST ? min(g, a.G - 1) * ST + s + 1 : gn * ST;
            load_x(next_stage, xbuf + (buf ^ 1) * XT);
            if (s == 0)
                load_group(gn, raw);
            __builtin_amdgcn_sched_barrier(0);
            const unsigned char *xt = xbuf + buf * XT;
            if (g <= g_last) {
                v8h B[2][RT], A[2][TT];
                auto decode = [&](int st, v8h *b) {
#pragma unroll
                    for (int q = 0; q < RT; ++q)
                        b[q] = __builtin_bit_cast(v8h, decode8<K>(masks, cur.tab[q], cur.pat[q][s * SPS + st]));
                };
                auto read = [&](int st, v8h *v) {
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt)
                        v[tt] = __builtin_bit_cast(v8h, *(const uint4 *)(xt + 32 * tt * (256 / ST) + x_step(st)));
                };
                read(0, A[0]);
                decode(0, B[0]);
#pragma unroll
                for (int st = 0; st < SPS; ++st) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (st + 1 < SPS) {
                        read(st + 1, A[(st + 1) & 1]);
                        decode(st + 1, B[(st + 1) & 1]);
                    }
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                        for (int q = 0; q < RT; ++q)
                            acc[q][tt] =
                                __builtin_amdgcn_mfma_f32_32x32x16_f16(A[st & 1][tt], B[st & 1][q], acc[q][tt], 0, 0, 0);
                    if (st + 1 < SPS) {
                        // the next step's operand reads behind the first
                        // product, a share of its decoding behind every one
#pragma unroll
                        for (int i = 0; i < TT * RT; ++i) {
                            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                            if (i == 0)
                                __builtin_amdgcn_sched_group_barrier(0x100, TT, 0);
                            __builtin_amdgcn_sched_group_barrier(0x2, 32 / TT, 0);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            buf ^= 1;
            sync();
        }
    }
    if constexpr (R == 1)
        __syncthreads();  // the sums below reuse every wavefront's tile
    // ---- the S K-slices of each row group summed in a fixed order (halving
    // tree through LDS; slot of K-slice s of row group rg: rg * S/2 + s) ----
    constexpr int NV = RT * TT * 16;  // values per lane
    float *red = (float *)smem;       // [R][S / 2][NV][64 lanes]
    for (int half = S / 2; half >= 1; half /= 2) {
        if (ks_id >= half && ks_id < 2 * half) {
            float *dst = red + ((size_t)rg * (S / 2) + (ks_id - half)) * (NV * 64);
#pragma unroll
            for (int q = 0; q < RT; ++q)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        dst[((q * TT + tt) * 16 + e) * 64 + lane] = acc[q][tt][e];
        }
        __syncthreads();
        if (ks_id < half) {
            const float *src = red + ((size_t)rg * (S / 2) + ks_id) * (NV * 64);
#pragma unroll
            for (int q = 0; q < RT; ++q)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        acc[q][tt][e] += src[((q * TT + tt) * 16 + e) * 64 + lane];
        }
        __syncthreads();
    }
    if (ks_id != 0)
        return;
#pragma unroll
    for (int q = 0; q < RT; ++q) {
        const int oo = o_base + 32 * q + n;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int t = t_base + 32 * tt + 8 * (e / 4) + 4 * kh + e % 4;
                if (oo < a.O && t < a.T)
                    a.Y[(size_t)t * a.O + oo] = __half_as_ushort(__float2half_rn(acc[q][tt][e]));
            }
    }
}


// Short prompts and small matrices (see the top of the file).
template <int K, int TT, int NW>
__global__ void __launch_bounds__(64 * NW) prefill_short_kernel(PrefillArgs a)
{
    constexpr int TR = tile_rows(K);
    constexpr unsigned PBLK_B = GB * TR * K * 16, CBLK_B = GB * TR * K * 2;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, w = wave_id();
    const int nw = blockDim.x >> 6;
    const int n = lane & 15, kq = lane >> 4;
    const int o_base = blockIdx.x * 16, t_base = blockIdx.y * 16 * TT;
    const int g0 = w * a.gps, g_end = min(g0 + a.gps, a.G);
    const int rows_dev = a.n_tiles * TR;

    v4f acc[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
        acc[tt] = v4f{0.f, 0.f, 0.f, 0.f};

    const int o = min(o_base + n, rows_dev - 1);
    const bool row_ok = o_base + n < rows_dev;
    const int r = o % TR;
    const unsigned blk = (unsigned)(o / TR) * (unsigned)a.n_gblocks;
    // lane quarter q loads plane q's slot (the last one where k < 4); a transpose
    // across the quarters then gives it word q of every plane
    const unsigned p_lane = blk * PBLK_B + (unsigned)(r * K + min(kq, K - 1)) * 16u;
    const unsigned c_lane = blk * CBLK_B + (unsigned)coeff_entry(K, r, 0, 0) * 2u;
    // activation tiles of the wavefront's K-slice, rows rounded up to four tokens
    const int x_inst = (min(16 * TT, a.T - t_base) + 3) / 4;
    const unsigned xt_bytes = (unsigned)((min(16 * TT, a.T) + 3) / 4) * 1024u;
    unsigned char *xbuf = smem + (size_t)w * 2 * xt_bytes;
    unsigned x_lane[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const int t = min(16 * tt + n, 4 * x_inst - 1);
        x_lane[tt] = (unsigned)(t * 256 + (((t & 15) ^ (4 * kq)) << 4));
    }
    auto load_x = [&](int g, unsigned char *buf) {
        for (int i = 0; i < x_inst; ++i) {
            const int t = 4 * i + (lane >> 4), c = (lane & 15) ^ (t & 15);
            load_to_lds(a.X + (size_t)min(t_base + t, a.T - 1) * a.I + (size_t)g * GROUP + c * 8, buf + i * 1024);
        }
    };
    uint4 slot;
    RowCoefs<K> coef;
    auto load_group = [&](int g) {
        const unsigned pu = (unsigned)(g / GB) * PBLK_B + (unsigned)(g % GB) * (TR * K * 16);
        const unsigned char *pb = (const unsigned char *)a.planes + pu;
        const unsigned char *cb = (const unsigned char *)a.coeffs + (unsigned)(g / GB) * CBLK_B;
        slot = *(const uint4 *)(pb + p_lane);
        coef = load_row_coefs<K>(cb + c_lane, g % GB);
    };
    DecodeMasks masks;
    masks.set();
    if (g0 < g_end) {
        load_x(g0, xbuf);
        load_group(g0);
        wait_loads();
        wave_sync();
        int buf = 0;
        for (int g = g0; g < g_end; ++g) {
            const int gn = min(g + 1, g_end - 1);
            const RowCoefs<K> c = row_coefs<K>(coef, g, row_ok);
            RowTable<K> tab = quarter_table32<K>(c, kq);
            if (__builtin_amdgcn_ballot_w64(!row_sums_exact_in_f32<K>(c)) != 0)
                tab = quarter_table64<K>(c, kq);
            const uint4 tw = transpose_rows4(slot);
            const uint32_t words[4] = {tw.x, tw.y, tw.z, tw.w};
            uint32_t pat[4];
            subset_indices<K>(masks, words, pat);
            load_x(gn, xbuf + (buf ^ 1) * xt_bytes);
            load_group(gn);
            __builtin_amdgcn_sched_barrier(0);
            const unsigned char *xt = xbuf + buf * xt_bytes;
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                v8h A[TT];
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
                    A[tt] = __builtin_bit_cast(v8h, *(const uint4 *)(xt + (x_lane[tt] ^ (st << 4))));
                const v8h B = __builtin_bit_cast(v8h, decode8<K>(masks, tab, pat[st]));
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
                    acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[tt], B, acc[tt], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            buf ^= 1;
            wait_loads();
            wave_sync();
        }
    }
    __syncthreads();
    // the K-slices' sums in slice order
    float *red = (float *)smem;  // [nw][TT * 4][64 lanes]
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            red[(w * (TT * 4) + tt * 4 + e) * 64 + lane] = acc[tt][e];
    __syncthreads();
    for (int idx = threadIdx.x; idx < TT * 4 * 64; idx += blockDim.x) {
        const int l = idx & 63, e = (idx >> 6) & 3, tt = idx >> 8;
        const int oo = o_base + (l & 15), t = t_base + 16 * tt + 4 * (l >> 4) + e;
        if (oo < a.O && t < a.T) {
            float s = 0.f;
            for (int q = 0; q < nw; ++q)
                s += red[q * (TT * 4 * 64) + idx];
            a.Y[(size_t)t * a.O + oo] = __half_as_ushort(__float2half_rn(s));
        }
    }
}

// Launch shapes.  prefill_kernel: rt, tt, r, st; prefill_short_kernel: rt = 0,
// tt, r = the most wavefronts.  cost: the time of a launch in microseconds.
// With f workgroups per CU (c = f rounded up), of which a CU holds `held` at
// once (LDS, wavefronts, registers; r = f / held rounded up: the rounds), and g
// groups per K-slice,
//   prefill_kernel        [0] + [1] g + ([2] c + [3] f + [5] r) g + [4] c + [6] r
//   prefill_short_kernel  [0] + [1] g + ([2] c + [3] f + [5] f x / 4) g n / 16
//                             + ([6] + [7] x) r g + [4] c + [8] r
// for n wavefronts and x loads of four tokens per group.  The shape with the
// lowest cost runs.
//
// Fitted on MI355X to the times of all twelve shapes on 6719 matrices and
// prompts (1 .. 28672 rows, 128 .. 28672 columns, 1 .. 2048 tokens, k = 1 .. 4,
// the sizes spread over their logarithms; each shape forced in turn, 2 to 40
// launches back to back over rotating weights): a non-negative least-squares
// fit of the relative error, then single steps of the constants that lower the
// time of the chosen shape over the best one's.  k is left out: constants of
// each k's own gained 0.1 %.  On 2757 further cases the choice takes 0.9 % more
// than the best shape on average (5.8 % at the 95th percentile, 24 % at most);
// a fit without the rounds (and with a shape less) took 2.7 % more, the present
// one is slower than it by over 3 % on 1.3 % of the cases (21 % at most).
// Against the LDS-table kernels it takes 0.65 / 0.58 / 0.54 / 0.56 of the time at
// k = 1 / 2 / 3 / 4 (geometric means over all 9476); 2 are slower by more than 2 %
// (15846 x 1408, k = 1, 16 tokens, 9 %; 163 x 5632, k = 1, 2038 tokens, 4 %).
// What the terms are for: without the rounds a shape that a CU holds once was
// taken for one that shares it (18332 x 896, k = 2, 23 tokens 16.2 us; 11.4 with
// the LDS tables, 8.5 with the best shape), and without the shape of 32 tokens
// and eight row groups matrices of one group took up to 1.29 times the LDS
// tables' time (6599 x 128, k = 1, 265 tokens 6.6 us instead of 4.1).
struct PrefillShape {
    int rt, tt, r, st;
    int held;  // prefill_kernel: workgroups a CU holds at once (the short kernel's: see prefill_cost)
    float cost[9];
};

static const PrefillShape PREFILL_SHAPES[] = {
    {0, 1, 8, 1, 0, {1.810f, 0.268f, 0.509f, 0.378f, 0.164f, 0.234f, 0.000f, 0.060f, 0.381f}},
    {0, 1, 16, 1, 0, {1.670f, 0.034f, 0.831f, 0.016f, 0.457f, 0.301f, 0.000f, 0.089f, 0.616f}},
    {0, 2, 8, 1, 0, {1.250f, 0.316f, 0.339f, 0.669f, 0.345f, 0.000f, 0.000f, 0.074f, 0.920f}},
    {1, 1, 1, 1, 1, {0.392f, 0.305f, 0.703f, 0.355f, 2.736f}},
    {1, 2, 1, 2, 1, {0.147f, 0.007f, 1.106f, 1.079f, 3.932f}},
    {1, 2, 2, 1, 1, {0.801f, 0.004f, 0.758f, 0.721f, 4.110f}},
    {1, 2, 4, 1, 2, {1.949f, 0.366f, 0.467f, 0.483f, 1.493f, 0.153f, 0.593f}},
    {1, 4, 2, 2, 1, {0.043f, 0.165f, 1.262f, 0.889f, 7.315f}},
    {1, 4, 4, 1, 1, {2.572f, 0.012f, 1.107f, 0.835f, 3.777f}},
    {1, 4, 8, 1, 1, {1.142f, 0.001f, 1.241f, 0.524f, 4.299f}},
    {1, 1, 8, 1, 2, {1.859f, 0.490f, 0.215f, 0.480f, 1.189f, 0.001f, 0.002f}},
    {2, 4, 8, 1, 1, {0.698f, 0.001f, 0.869f, 2.719f, 9.087f}},
};

// LDS of a launch: two activation stages per K-slice, which the partial sums
// then reuse.
static size_t prefill_lds(const PrefillShape &s, int T, int slices)
{
    const size_t stages = s.rt ? (size_t)slices * 2 * (32 * s.tt * GROUP * 2 / s.st)
                               : (size_t)slices * 2 * ((min(T, 16 * s.tt) + 3) / 4) * 1024;
    const size_t sums = s.rt ? (size_t)s.r * (slices / 2) * s.rt * s.tt * 16 * 64 * 4
                             : (size_t)slices * s.tt * 4 * 64 * 4;
    return stages > sums ? stages : sums;
}

static double prefill_cost(const PrefillShape &s, const Dims &d, int T, int slices, double wg)
{
    const double f = wg / PF_CUS, g = (d.G + slices - 1) / slices;
    // short kernel: at most 64 registers, so 32 wavefronts per CU
    const int held = s.rt ? s.held : max(1, min((int)(PF_LDS_MAX / prefill_lds(s, T, slices)), 32 / slices));
    const double c = ceil(f), r = ceil(f / held);
    const float *k = s.cost;
    if (s.rt)
        return k[0] + k[1] * g + (k[2] * c + k[3] * f + k[5] * r) * g + k[4] * c + k[6] * r;
    const double x = (min(T, 16 * s.tt) + 3) / 4;
    return k[0] + k[1] * g + (k[2] * c + k[3] * f + k[5] * f * x / 4) * g * slices / 16 +
           (k[6] + k[7] * x) * r * g + k[4] * c + k[8] * r;
}

template <int K>
static const void *prefill_kernel_for(const PrefillShape &s)
{
    if (s.rt == 0)
        return s.r > PF_WAVES ? (const void *)prefill_short_kernel<K, 1, 16>
               : s.tt == 1    ? (const void *)prefill_short_kernel<K, 1, 8>
                              : (const void *)prefill_short_kernel<K, 2, 8>;
    if (s.rt == 2)
        return (const void *)prefill_kernel<K, 2, 4, 8, 1>;
    if (s.tt == 1)
        return s.r == 1 ? (const void *)prefill_kernel<K, 1, 1, 1, 1> : (const void *)prefill_kernel<K, 1, 1, 8, 1>;
    if (s.tt == 2)
        return s.r == 1   ? (const void *)prefill_kernel<K, 1, 2, 1, 2>
               : s.r == 2 ? (const void *)prefill_kernel<K, 1, 2, 2, 1>
                          : (const void *)prefill_kernel<K, 1, 2, 4, 1>;
    return s.r == 2   ? (const void *)prefill_kernel<K, 1, 4, 2, 2>
           : s.r == 4 ? (const void *)prefill_kernel<K, 1, 4, 4, 1>
                      : (const void *)prefill_kernel<K, 1, 4, 8, 1>;
}

// The launch of a call: its shape (null: none can take it), K-slices and grid.
struct PrefillLaunch {
    const PrefillShape *shape;
    int slices, gx, gy;
};

static PrefillLaunch prefill_launch(const Dims &d, int T)
{
    PrefillLaunch best = {};
    double best_cost = 0;
    for (const PrefillShape &s : PREFILL_SHAPES) {
        const int sl = s.rt ? PF_WAVES / s.r : min(s.r, d.G);
        const int rows = s.rt ? 32 * s.rt * s.r : 16, tokens = s.rt ? 32 * s.tt : 16 * s.tt;
        const int x = (d.O + rows - 1) / rows, y = (T + tokens - 1) / tokens;
        if (y > 65535)  // (a grid's second dimension has 16 bits)
            continue;
        const double cost = prefill_cost(s, d, T, sl, (double)x * y);
        if (!best.shape || cost < best_cost) {
            best = {&s, sl, x, y};
            best_cost = cost;
        }
    }
    return best;
}

int launch_prefill(const Dims &d, const void *planes_dev, const void *coeffs_dev, const uint16_t *X, uint16_t *Y,
                   int T, hipStream_t stream)
{
    const PrefillLaunch l = prefill_launch(d, T);
    if (!l.shape)
        return SBVR_E_UNSUPPORTED;
    PrefillArgs a = {(const uint32_t *)planes_dev, (const uint16_t *)coeffs_dev, X, Y, d.O, d.I, T, d.n_tiles,
                     d.n_gblocks, d.G, (d.G + l.slices - 1) / l.slices};
    const size_t lds = prefill_lds(*l.shape, T, l.slices);
    if (lds > PF_LDS_MAX)
        return SBVR_E_UNSUPPORTED;
    const int waves = l.shape->rt ? PF_WAVES : l.slices;
    const void *fn = d.k == 4   ? prefill_kernel_for<4>(*l.shape)
                     : d.k == 3 ? prefill_kernel_for<3>(*l.shape)
                     : d.k == 2 ? prefill_kernel_for<2>(*l.shape)
                                : prefill_kernel_for<1>(*l.shape);
    void *args[] = {&a};
    return launch_kernel(fn, dim3(l.gx, l.gy), dim3(64 * waves), lds, stream, args);
}

}  // namespace sbvr

// Which launch shape a call takes, its index in PREFILL_SHAPES (-1: none), and
// how many shapes there are: for the tests, not part of the C ABI.
extern "C" int sbvr_test_prefill_shape(int O, int I, int k, int T)
{
    const sbvr::PrefillShape *s = sbvr::prefill_launch(sbvr::make_dims(O, I, k), T).shape;
    return s ? (int)(s - sbvr::PREFILL_SHAPES) : -1;
}

extern "C" int sbvr_test_prefill_shapes(void)
{
    return (int)(sizeof(sbvr::PREFILL_SHAPES) / sizeof(sbvr::PREFILL_SHAPES[0]));
}
