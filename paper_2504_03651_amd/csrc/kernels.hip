// kernels.hip -- gfx950 kernels of the mixed paged-attention iteration.
//
//   append_kernel       scatter new K/V into the paged pool (bf16 bit copy,
//                       or e4m3 quantisation with per-(block, head) scales)
//   block_copy_kernel   whole-block copy-on-write
//   attn_kernel         one wave per (work descriptor, KV head, head chunk): up
//                       to 16 query vectors against a run of 16-token blocks,
//                       online softmax, bf16 MFMA
//   merge_kernel        log-sum-exp merge of split / segment partial results
//
// MFMA tile orientation (v_mfma_f32_16x16x32_bf16, wave64):
//   S^T[key][query] = K[key][d] * Q^T[d][query]     (keys on rows)
//   O^T[d][query]  += V^T[d][key] * P^T[key][query]
// so each lane ends up owning one query column and the softmax statistics of
// that query never leave the lane's 16-lane column group.  K blocks are stored
// [16][D] and V blocks [D][16], which makes every MFMA operand a contiguous
// load straight from the pool (16 bytes, or 8 for e4m3 V).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <stdint.h>
#include <type_traits>

#include "kernels.hpp"

namespace echo {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// P.V products: bf16 (bf16 cache) or fp16 (e4m3 cache) operands, fp32 accumulate
__device__ __forceinline__ f32x4_t mfma_pv(bf16x8_t a, bf16x8_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4_t mfma_pv(f16x8_t a, f16x8_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------- codecs

// OCP e4m3fn -> bf16, exact (every e4m3 value is a bf16 value): gfx950's
// v_cvt_scalef32_pk_bf16_fp8 with scale 1 widens two codes per instruction
// (checked on all 256 codes, NaN and signed zero included).
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16x8_t e4m3x8_to_bf16x8(u32x2_t w) {
    const bf16x2_t a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[0], 1.0f, false);
    const bf16x2_t b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[0], 1.0f, true);
    const bf16x2_t c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[1], 1.0f, false);
    const bf16x2_t d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[1], 1.0f, true);
    return (bf16x8_t){a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
}

// Two fp32 -> two OCP e4m3fn codes in the low 16 bits, round to nearest even,
// saturating to +-448, NaN to 0x7F: gfx950's v_cvt_pk_fp8_f32 on the clamped
// values (the tests compare the codes of every bf16 value, at scales inside and
// outside the quotient's fast range, with the oracle's encoder).
__device__ __forceinline__ uint32_t f32x2_to_e4m3(float x, float y) {
    const uint32_t w = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(
        __builtin_amdgcn_fmed3f(x, -448.f, 448.f), __builtin_amdgcn_fmed3f(y, -448.f, 448.f), 0, false);
    const uint32_t nan = (x != x ? 0x7Fu : 0u) | (y != y ? 0x7F00u : 0u);
    const uint32_t keep = (x != x ? 0u : 0xFFu) | (y != y ? 0u : 0xFF00u);
    return (w & keep) | nan;
}

// The quotient RN(x / s) that the quantisation takes, for a divisor s shared
// by a whole (block, head) tile: from r = RN(1 / s), q0 = RN(x r), the exact
// residual e = x - q0 s (one FMA) and the corrected q1 = RN(q0 + e r)
// (Markstein's final correction step).  For s in [2^-100, 2^100] this gives
// the same e4m3 code as the correctly rounded quotient for every finite bf16
// x (checked exhaustively on the CPU over x and every scale fp32(b / 448), b
// a positive bf16); quotients past 512 saturate either way and keep q0, and
// the sign is q0's (a zero x keeps its sign).  Other scales divide.
// The scale is the wave's, so it is kept scalar and the choice is one branch.
struct Recip {
    float s, r;
    bool fast;
};
__device__ __forceinline__ float uniform(float x) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}
__device__ __forceinline__ Recip recip_of(float s) {
    s = uniform(s);
    return {s, uniform(1.0f / s), s >= 0x1p-100f && s <= 0x1p100f};
}
template <bool FAST>
__device__ __forceinline__ float quotient(float x, const Recip &d) {
    if constexpr (!FAST) return x / d.s;
    const float q0 = x * d.r;
    const float e = __builtin_fmaf(-q0, d.s, x);
    const float q1 = __builtin_fmaf(e, d.r, q0);
    return __builtin_copysignf(__builtin_fabsf(q0) < 512.0f ? q1 : q0, q0);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// v_max_f32 as such: fmaxf adds a canonicalising max of each operand the
// compiler cannot prove canonical (lane-swap results are not), two extra VALU
// ops per call.  Used on attention scores, which are finite or -inf.
__device__ __forceinline__ float vmax(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
// max over lanes l, l^16, l^32, l^48 with VALU lane swaps (no LDS traffic):
// each swap returns the lane's own value and its partner's, in some order.
__device__ __forceinline__ float wave_max_xor16_32(float x) {
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    const u2 a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = vmax(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const u2 b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return vmax(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// ------------------------------------------------------------------- append

// One work unit = (row, written block, KV head), one wave each.  Bound by
// memory latency and by how the accesses coalesce, so a block goes through the
// wave in 16-byte pieces both ways: lane (a, c) holds the 16-byte chunk c of
// slots SL * a .. + SL (SL = D / 32), so that every load and every K store of
// the wave covers whole rows; V's SL slots x 8 values are transposed in
// registers, and the wave's LDS tile turns them into whole 1 KiB runs of the
// [d][16 slots] tile.  A block written in part (a decode row's slot, a chunk's
// ends) reads its V tile beside the new tokens and writes it back whole: the
// L2 would fetch those lines for 2-byte stores as well.  9,924 prompt tokens
// (8 KV heads, head_dim 64, bf16): 27 -> 10 us, 4 TB/s; 16,412 tokens at
// head_dim 128: 35 -> 27 us, 5 TB/s; 4,640 tokens of 546 rows into an e4m3
// cache: 28.7 -> 16.7 us; 256 decode rows of 32 heads: 17.2 -> 15.6 us.

// Codes of eight bf16 values, in order
template <bool FAST>
__device__ __forceinline__ u32x2_t e4m3x8_by(const u32x4_t &w, const Recip &d) {
    u32x2_t c;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        uint32_t h[2];
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const uint32_t v = w[2 * x + y];
            h[y] = f32x2_to_e4m3(quotient<FAST>(bf16_bits_to_f32(v & 0xFFFFu), d),
                                 quotient<FAST>(bf16_bits_to_f32(v >> 16), d));
        }
        c[x] = h[0] | (h[1] << 16);
    }
    return c;
}
__device__ __forceinline__ u32x2_t e4m3x8(const u32x4_t &w, const Recip &d) {
    return d.fast ? e4m3x8_by<true>(w, d) : e4m3x8_by<false>(w, d);
}

// byte i of the result: byte (sel >> 8i & 7) of the pair (hi: 4..7, lo: 0..3)
__device__ __forceinline__ uint32_t bytes(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

__device__ __forceinline__ float absmax8(const u32x4_t &w, float m) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
        m = fmaxf(m, fmaxf(fabsf(bf16_bits_to_f32(w[x] & 0xFFFFu)), fabsf(bf16_bits_to_f32(w[x] >> 16))));
    return m;
}

__device__ __forceinline__ float wave_max(float m) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    return m;
}

// LDS of one wave's V tile: rows d of 16 slots, 8 rows and a pad per chunk
// (the pad spreads the chunks over the banks)
template <int D, bool FP8>
struct AppendTile {
    static constexpr int ROW = FP8 ? 16 : 32;              // bytes
    static constexpr int CHUNK = 8 * ROW + (FP8 ? 16 : 32);
    static constexpr int BYTES = D / 8 * CHUNK;
};

// Slots m0 .. m0 + n - 1 of block blk, head h, from tokens t .. t + n - 1.
template <int D, bool FP8>
__device__ __forceinline__ void append_block(const AppendArgs &a, int blk, int h, int64_t t, int m0,
                                             int n, int lane, uint8_t *lds) {
    typedef AppendTile<D, FP8> TL;
    constexpr int SL = D / 32, CH = D / 8;   // slots per lane, 16-byte chunks per row
    constexpr int NU = D * TL::ROW / 1024;   // 1 KiB runs of the V tile
    const int c = lane % CH, s0 = SL * (lane / CH);
    const int64_t H = a.num_kv_heads, src = (t + s0 - m0) * H * D + (int64_t)h * D + 8 * c;
    const int64_t tile = ((int64_t)blk * H + h) * 16 * D;
    const bool full = n == 16;
    bool mine[SL];
    u32x4_t kw[SL], vw[SL], old[NU];
#pragma unroll
    for (int w = 0; w < SL; ++w) {
        mine[w] = (uint32_t)(s0 + w - m0) < (uint32_t)n;
        kw[w] = vw[w] = (u32x4_t){0u, 0u, 0u, 0u};
        if (mine[w]) {
            kw[w] = *(const u32x4_t *)(a.k_new + src + w * H * D);
            vw[w] = *(const u32x4_t *)(a.v_new + src + w * H * D);
        }
    }
    uint8_t *vdst = (uint8_t *)a.v + tile * (FP8 ? 1 : 2) + 16 * lane;
    if (!full) {
#pragma unroll
        for (int i = 0; i < NU; ++i) old[i] = *(const u32x4_t *)(vdst + i * 1024);
    }
    uint8_t *vl = lds + c * TL::CHUNK + s0 * (FP8 ? 1 : 2);
    if constexpr (!FP8) {
        uint16_t *kdst = (uint16_t *)a.k + tile + s0 * D + 8 * c;
#pragma unroll
        for (int w = 0; w < SL; ++w)
            if (mine[w]) *(u32x4_t *)(kdst + w * D) = kw[w];
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int e = 0; e < 2; ++e) {   // d = 8c + 2x + e
                const uint32_t sel = e ? 0x07060302u : 0x05040100u;
                uint8_t *row = vl + (2 * x + e) * TL::ROW;
                if constexpr (SL == 4)
                    *(u32x2_t *)row = (u32x2_t){bytes(vw[1][x], vw[0][x], sel),
                                                bytes(vw[SL - 1][x], vw[SL - 2][x], sel)};
                else
                    *(uint32_t *)row = bytes(vw[1][x], vw[0][x], sel);
            }
    } else {
        const int64_t si = (int64_t)blk * H + h;
        float sk, sv;
        if (m0 == 0) {   // slot 0 written by this call: fresh scales
            float ak = 0.f, av = 0.f;
#pragma unroll
            for (int w = 0; w < SL; ++w) {
                ak = absmax8(kw[w], ak);
                av = absmax8(vw[w], av);
            }
            ak = wave_max(ak);
            av = wave_max(av);
            sk = ak == 0.f ? 1.f : ak / 448.0f;
            sv = av == 0.f ? 1.f : av / 448.0f;
            if (lane == 0) {
                a.k_scale[si] = sk;
                a.v_scale[si] = sv;
            }
        } else {
            sk = a.k_scale[si];
            sv = a.v_scale[si];
        }
        const Recip dk = recip_of(sk), dv = recip_of(sv);
        uint8_t *kdst = (uint8_t *)a.k + tile + s0 * D + 8 * c;
        u32x2_t vc[SL];
#pragma unroll
        for (int w = 0; w < SL; ++w) {
            vc[w] = (u32x2_t){0u, 0u};
            if (mine[w]) {   // one slot of a decode row: the other SL - 1 are skipped
                *(u32x2_t *)(kdst + w * D) = e4m3x8(kw[w], dk);
                vc[w] = e4m3x8(vw[w], dv);
            }
        }
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            // 4 values x SL slots of bytes, transposed
            const uint32_t p01 = bytes(vc[1][x], vc[0][x], 0x05010400u);   // d0: s0 s1, d1: s0 s1
            const uint32_t q01 = bytes(vc[1][x], vc[0][x], 0x07030602u);   // d2, d3
            if constexpr (SL == 4) {
                const uint32_t p23 = bytes(vc[SL - 1][x], vc[SL - 2][x], 0x05010400u);
                const uint32_t q23 = bytes(vc[SL - 1][x], vc[SL - 2][x], 0x07030602u);
                *(uint32_t *)(vl + (4 * x + 0) * TL::ROW) = bytes(p23, p01, 0x05040100u);
                *(uint32_t *)(vl + (4 * x + 1) * TL::ROW) = bytes(p23, p01, 0x07060302u);
                *(uint32_t *)(vl + (4 * x + 2) * TL::ROW) = bytes(q23, q01, 0x05040100u);
                *(uint32_t *)(vl + (4 * x + 3) * TL::ROW) = bytes(q23, q01, 0x07060302u);
            } else {
                *(uint16_t *)(vl + (4 * x + 0) * TL::ROW) = (uint16_t)p01;
                *(uint16_t *)(vl + (4 * x + 1) * TL::ROW) = (uint16_t)(p01 >> 16);
                *(uint16_t *)(vl + (4 * x + 2) * TL::ROW) = (uint16_t)q01;
                *(uint16_t *)(vl + (4 * x + 3) * TL::ROW) = (uint16_t)(q01 >> 16);
            }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // this lane's 16-byte units of the V tile hold slots u0 ..: all 16 of a
    // row (e4m3) or half of them; those written now come from LDS
    const int u0 = FP8 ? 0 : 8 * (lane & 1);
    constexpr int PER = FP8 ? 4 : 2;   // slots per 32-bit word
    u32x4_t keep;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        uint32_t m = 0;
#pragma unroll
        for (int y = 0; y < PER; ++y)
            if ((uint32_t)(u0 + PER * x + y - m0) >= (uint32_t)n)
                m |= (FP8 ? 0xFFu : 0xFFFFu) << (32 / PER * y);
        keep[x] = m;
    }
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int off = i * 1024 + 16 * lane;   // bytes into the tile
        u32x4_t v = *(const u32x4_t *)(lds + off / (8 * TL::ROW) * TL::CHUNK + off % (8 * TL::ROW));
        if (!full) v = (v & ~keep) | (old[i] & keep);
        *(u32x4_t *)(vdst + i * 1024) = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Block j of row r, whose first new token is t0 at position p0 of L.
template <int D, bool FP8>
__device__ __forceinline__ void append_unit(const AppendArgs &a, int r, int j, int h, int t0, int p0,
                                            int L, int lane, uint8_t *lds) {
    if (j >= a.max_blocks_per_row) return;
    const int blk = a.block_tables[(int64_t)r * a.max_blocks_per_row + j];
    if (blk < 0 || blk >= a.num_blocks) return;
    const int lo = max(p0, 16 * j), n = min(L, 16 * j + 16) - lo;   // tokens written
    append_block<D, FP8>(a, blk, h, (int64_t)t0 + (lo - p0), lo & 15, n, lane, lds);
}

// A row of q new tokens writes at most q / 16 + 2 blocks, so with its units
// numbered from q_start / 16 + 2 row no two rows' numbers meet, and a wave
// finds the row of its number from q_start alone: 64 rows probed per load.
// No scan, no barrier: rows of any mix of lengths take T / 16 + 2 B waves per
// head, and a wave waits for one load (two past 64 rows) more than in the
// direct form below.  (With a scan of all rows in every workgroup the e4m3
// batch above took 25.4 us; with a loop over units, whose hoisted addresses
// cost a wave per SIMD, 18.3 us.)
template <int D, bool FP8>
__global__ __launch_bounds__(256) void append_kernel(AppendArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t vstage[4][AppendTile<D, FP8>::BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t unit = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 4 + wave;
    if (unit >= a.n_units) return;
    const uint32_t H = a.num_kv_heads;
    const int B = a.num_rows;
    const int64_t u = unit >> 32 ? unit / H : (int64_t)((uint32_t)unit / H);
    const int h = (int)(unit - u * H);
    int r = 0;   // last row whose numbers start at or before u
    for (int n = B;;) {
        const int step = (n + 63) >> 6, i = r + lane * step;
        const bool at = lane * step < n && (int64_t)(a.q_start[i < B ? i : 0] >> 4) + 2 * (int64_t)i <= u;
        const int k = max(__popcll(__ballot(at)), 1) - 1;
        r += k * step;
        if (step == 1) break;
        n = min(step, n - k * step);
    }
    r = __builtin_amdgcn_readfirstlane(r);
    const int t0 = a.q_start[r];
    const int q = a.q_start[r + 1] - t0;
    const int L = a.seq_lens[r];
    const int p0 = L - q;
    const int64_t k = u - ((t0 >> 4) + 2 * (int64_t)r);
    if (q <= 0 || p0 < 0 || k < 0 || k > (L - 1) / 16 - p0 / 16) return;
    append_unit<D, FP8>(a, r, p0 / 16 + (int)k, h, t0, p0, L, lane, vstage[wave]);
}

// Direct form for batches whose rows write about as many blocks each (decode
// rows above all): one wave per (row, k-th written block, KV head).
template <int D, bool FP8>
__global__ __launch_bounds__(256) void append_rows_kernel(AppendArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t vstage[4][AppendTile<D, FP8>::BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t unit = blockIdx.x * 4u + wave;
    if (unit >= (uint32_t)a.n_units) return;
    const uint32_t H = a.num_kv_heads, bpr = a.blocks_per_row;
    const uint32_t rest = unit / H;
    const int h = (int)(unit - rest * H);
    const int r = (int)(rest / bpr), k = (int)(rest - (rest / bpr) * bpr);
    const int t0 = a.q_start[r];
    const int q = a.q_start[r + 1] - t0;
    const int L = a.seq_lens[r];
    const int p0 = L - q;
    if (q <= 0 || p0 < 0) return;
    const int j = p0 / 16 + k;
    if (j > (L - 1) / 16) return;
    append_unit<D, FP8>(a, r, j, h, t0, p0, L, lane, vstage[wave]);
}

// --------------------------------------------------------------- block copy

__global__ __launch_bounds__(256) void block_copy_kernel(BlockCopyArgs a) {
    const int64_t unit = blockIdx.x;
    const int pair = (int)(unit / a.chunks);
    const int chunk = (int)(unit % a.chunks);
    if (pair >= a.n_pairs) return;
    const int src = a.pairs[2 * pair], dst = a.pairs[2 * pair + 1];
    if (src < 0 || src >= a.num_blocks || dst < 0 || dst >= a.num_blocks) return;
    const int64_t words = a.block_bytes / 16;
    const u32x4_t *ks = (const u32x4_t *)((const uint8_t *)a.k + (int64_t)src * a.block_bytes);
    const u32x4_t *vs = (const u32x4_t *)((const uint8_t *)a.v + (int64_t)src * a.block_bytes);
    u32x4_t *kd = (u32x4_t *)((uint8_t *)a.k + (int64_t)dst * a.block_bytes);
    u32x4_t *vd = (u32x4_t *)((uint8_t *)a.v + (int64_t)dst * a.block_bytes);
    // Every load before the first store: the compiler cannot know that blocks
    // do not overlap, and one load at a time leaves the memory idle.  The copy
    // is not read soon, so its stores pass the L2 by, which keeps the lines of
    // the sources: 1,024 blocks of 64 KiB (K and V) 32.0 -> 27.1 us, 5 TB/s
    // (ordinary stores 33.5 us, non-temporal loads alone 27.2, both 29.5).
    u32x4_t kw[4], vw[4];
    const int64_t base = (int64_t)chunk * 1024;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t w = base + e * 256 + threadIdx.x;
        kw[e] = vw[e] = (u32x4_t){0u, 0u, 0u, 0u};
        if (w < words) {
            kw[e] = ks[w];
            vw[e] = vs[w];
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t w = base + e * 256 + threadIdx.x;
        if (w < words) {
            __builtin_nontemporal_store(kw[e], kd + w);
            __builtin_nontemporal_store(vw[e], vd + w);
        }
    }
    if (a.k_scale && chunk == 0) {
        for (int h = threadIdx.x; h < a.num_kv_heads; h += 256) {
            a.k_scale[(int64_t)dst * a.num_kv_heads + h] = a.k_scale[(int64_t)src * a.num_kv_heads + h];
            a.v_scale[(int64_t)dst * a.num_kv_heads + h] = a.v_scale[(int64_t)src * a.num_kv_heads + h];
        }
    }
}

// ---------------------------------------------------------------- attention

// Read-only metadata (work descriptors, block tables) through the constant
// address space: nothing writes it while a kernel runs, so wave-uniform reads
// are scalar loads wherever they sit in the kernel.
typedef const __attribute__((address_space(4))) int32_t const_i32;
__device__ __forceinline__ int32_t ro_load(const int32_t *p, int64_t i) {
    return ((const_i32 *)p)[i];
}

// Pool loads: streamed past the L2 (non-temporal) when no other wave reads
// the same keys, ordinary otherwise.
template <bool B>
struct Flag {
    static constexpr bool value = B;
};
template <bool NT, typename R>
__device__ __forceinline__ R pool_load(const void *p) {
    if constexpr (NT) return __builtin_nontemporal_load((const R *)p);
    else return *(const R *)p;
}

// Per-dtype pieces of the decode kernel.  A lane's K operand for the 32-wide
// contraction chunk c is 8 values of d; which 8 is free as long as Q uses the
// same assignment.  bf16 takes d = 32c + 8*g4 (one 16-byte load per chunk);
// e4m3 takes d = 64(c/2) + 16*g4 + 8(c%2), so one 16-byte load of 16 codes
// feeds two chunks and every K load is 16 bytes wide for both dtypes.
template <bool FP8>
struct KV;
template <>
struct KV<false> {
    typedef uint16_t T;
    typedef u32x4_t VRaw;                   // 8 keys of one V^T row
    static constexpr int KSTEP = 32;        // elements between a lane's K loads
    static constexpr int KLANE = 8;         // elements per 16-lane group and load
    static __device__ __forceinline__ int q_off(int c, int g4) { return 32 * c + 8 * g4; }
    static __device__ __forceinline__ bf16x8_t k_chunk(const u32x4_t *kr, int c) {
        return __builtin_bit_cast(bf16x8_t, kr[c]);
    }
    static __device__ __forceinline__ bf16x8_t widen(VRaw r) { return __builtin_bit_cast(bf16x8_t, r); }
    // zero element e (0..7) where bit e of keep is clear
    static __device__ __forceinline__ VRaw mask(VRaw r, uint32_t keep) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t m = ((keep >> (2 * w)) & 1u ? 0x0000FFFFu : 0u) |
                               ((keep >> (2 * w + 1)) & 1u ? 0xFFFF0000u : 0u);
            r[w] &= m;
        }
        return r;
    }
};
template <>
struct KV<true> {
    typedef uint8_t T;
    typedef u32x2_t VRaw;                   // 8 e4m3 keys of one V^T row
    static constexpr int KSTEP = 64;
    static constexpr int KLANE = 16;
    static __device__ __forceinline__ int q_off(int c, int g4) {
        return 64 * (c >> 1) + 16 * g4 + 8 * (c & 1);
    }
    static __device__ __forceinline__ bf16x8_t k_chunk(const u32x4_t *kr, int c) {
        const u32x4_t w = kr[c >> 1];
        return e4m3x8_to_bf16x8((c & 1) ? (u32x2_t){w[2], w[3]} : (u32x2_t){w[0], w[1]});
    }
    static __device__ __forceinline__ bf16x8_t widen(VRaw r) { return e4m3x8_to_bf16x8(r); }
    static __device__ __forceinline__ VRaw mask(VRaw r, uint32_t keep) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            uint32_t m = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) m |= ((keep >> (4 * w + b)) & 1u) ? (0xFFu << (8 * b)) : 0u;
            r[w] &= m;
        }
        return r;
    }
};

// Logical workgroup of physical workgroup P.  Workgroups are dispatched to
// the 8 XCDs round-robin (P mod 8); this order gives each XCD runs of
// 2^run_log2 consecutive logical workgroups, so the sibling waves of a shared
// segment (consecutive descriptors) read its blocks through one L2.  Runs are
// dealt to the XCDs in rounds of 8, in reverse order every other round: the
// work list is sorted heavy-first, so a plain round-robin deal would give XCD 0
// the heaviest run of every round (5-10% more work than XCD 7 on the batches
// measured) and the kernel would end when XCD 0 does.  Runs are 16 workgroups,
// shorter on small grids so that every XCD gets several.  The grid is a
// multiple of 8 runs, so the map is a permutation of the grid.
__device__ __forceinline__ int dec_logical(int P, int run_log2) {
    const int q = P >> 3, x = P & 7;
    const int round = q >> run_log2;
    const int xr = (round & 1) ? 7 - x : x;
    return ((round * 8 + xr) << run_log2) + (q & ((1 << run_log2) - 1));
}

// One decode workgroup of four waves: P is its physical workgroup index in
// the decode order (dec_logical), tid its thread index in [0, 256).
// Decode waves are bound by the CU's texture address units, and the SIMD
// issues the oldest ready wave first, so of three resident waves the oldest
// streams about twice as fast as the youngest.  Each wave therefore sets its
// issue priority from the 32-key steps it has left (longest remaining work
// first), which evens out the end times the planner assumes equal.
#ifndef ECHO_DEC_PRIO
#define ECHO_DEC_PRIO 24, 12, 6
#endif
constexpr int kDecPrio[3] = {ECHO_DEC_PRIO};   // steps left for priority 3, 2, 1

template <int D, bool FP8>
__device__ __forceinline__ void decode_body(const AttnArgs &a, int P, int tid) {
    typedef KV<FP8> kv;
    typedef typename kv::T KT;
    typedef typename kv::VRaw VRaw;
    constexpr int NC = D / 32;            // 32-wide d chunks of the QK contraction
    constexpr int NT = D / 16;            // 16-row d tiles of O^T
    constexpr int NK = D / kv::KSTEP;     // 16-byte K loads per key row and lane

    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t idx = (int64_t)dec_logical(P, a.run_log2) * 4 + wave;
    if (idx >= a.n_waves) return;
    if (a.counts && idx >= (int64_t)ro_load(a.counts, kHdrDesc) * a.waves_per_desc) return;
    const int di = (int)(idx / a.waves_per_desc);
    const int rem = (int)(idx - (int64_t)di * a.waves_per_desc);
    const int kvh = rem / a.head_chunks;
    const int hc = rem - kvh * a.head_chunks;
    const int32_t *ip = (const int32_t *)(a.desc + di);
    const int tok_off = __builtin_amdgcn_readfirstlane(ro_load(ip, 0));
    const int shape = __builtin_amdgcn_readfirstlane(ro_load(ip, 1));
    const int bt_row = __builtin_amdgcn_readfirstlane(ro_load(ip, 2));
    const int key_begin = __builtin_amdgcn_readfirstlane(ro_load(ip, 3));
    const int key_end = __builtin_amdgcn_readfirstlane(ro_load(ip, 4));
    const int dpart = __builtin_amdgcn_readfirstlane(ro_load(ip, 5));
    const int tok1 = __builtin_amdgcn_readfirstlane(ro_load(ip, 6));
    const int klim1 = __builtin_amdgcn_readfirstlane(ro_load(ip, 7));
    const int nt = shape & 0xFF;
    const int h0 = kvh * a.group + hc * 16;
    const int nh = min(a.heads_per_chunk, a.group - hc * 16);
    const int part = dpart < 0 ? -1 : dpart + rem * nt * a.heads_per_chunk;

    const int g4 = lane >> 4;   // 16-lane group: selects 8 of each 32 k-values
    const int c16 = lane & 15;  // MFMA row (A) / column (B, C) index
    const int qi = c16 / nh, qj = c16 - (c16 / nh) * nh;
    const bool qvalid = qi < nt;
    int tok = 0, klim = 0;
    if (qvalid) {
        if (nt == 1) {   // single-token slice: token and key limit ride in the descriptor
            tok = tok1;
            klim = klim1;
        } else {
            tok = a.tok_list[tok_off + qi];
            klim = a.klim[tok];
        }
    }
    const int head = h0 + qj;

    // Q^T as the B operand: column c16, the 8 d values kv::q_off(c, g4) ..
    bf16x8_t qf[NC];
    {
        const uint16_t *qp = a.q + ((int64_t)tok * a.num_q_heads + head) * D;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            u32x4_t w = {0u, 0u, 0u, 0u};
            if (qvalid) w = *(const u32x4_t *)(qp + kv::q_off(c, g4));
            qf[c] = __builtin_bit_cast(bf16x8_t, w);
        }
    }

    f32x4_t acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    const int32_t *btr = a.block_tables + (int64_t)bt_row * a.max_blocks_per_row;
    const int64_t blk_stride = (int64_t)a.num_kv_heads * 16 * D;
    const KT *kbase = (const KT *)a.k + (int64_t)kvh * 16 * D;
    const KT *vbase = (const KT *)a.v + (int64_t)kvh * 16 * D;
    // S^T tile t, row c16 holds key 8*(c16>>2) + 4t + (c16&3) of the 32-key
    // window, so lane (g4, c16) receives keys 8*g4 .. 8*g4+7 of its column.
    const int ksel = c16 >= 8;
    const int kslot = 8 * ((c16 >> 2) & 1) + (c16 & 3);
    // V^T tile i, row c16 is d = 16i + c16; k-values are keys 8*g4 .. +8
    const int vsel = g4 >= 2;
    const int vslot = 8 * (g4 & 1);
    const float scale = a.scale_log2;

    auto sweep = [&](auto nt_flag) {
        constexpr bool NTL = decltype(nt_flag)::value;
        for (int kb = key_begin; kb < key_end; kb += 32) {
            const int left = (key_end - kb + 31) >> 5;
            if (left >= kDecPrio[0]) __builtin_amdgcn_s_setprio(3);
            else if (left >= kDecPrio[1]) __builtin_amdgcn_s_setprio(2);
            else if (left >= kDecPrio[2]) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
            const int jb = kb >> 4;
            const int b0 = ro_load(btr, jb);
            const bool has1 = kb + 16 < key_end;
            const int b1 = has1 ? ro_load(btr, jb + 1) : b0;
            const int kblk = ksel ? b1 : b0;
            const int vblk = vsel ? b1 : b0;

            u32x4_t kr[2][NK];
            VRaw vr[NT];
            const KT *kp = kbase + (int64_t)kblk * blk_stride + kslot * D + kv::KLANE * g4;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int p = 0; p < NK; ++p)
                    kr[t][p] = pool_load<NTL, u32x4_t>(kp + 4 * t * D + kv::KSTEP * p);
            const KT *vp = vbase + (int64_t)vblk * blk_stride + c16 * 16 + vslot;
#pragma unroll
            for (int i = 0; i < NT; ++i) vr[i] = pool_load<NTL, VRaw>(vp + i * 256);
            // every K and V load of the step goes out before the products (left
            // to itself the compiler reuses K's registers for V and issues the
            // V loads only after the first K values arrive)
            __builtin_amdgcn_sched_barrier(0);

            f32x4_t s[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                s[t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kv::k_chunk(kr[t], c), qf[c],
                                                                   s[t], 0, 0, 0);
            }

            float sk = scale, sv = 1.f;
            if constexpr (FP8) {
                sk = scale * a.k_scale[(int64_t)vblk * a.num_kv_heads + kvh];
                sv = a.v_scale[(int64_t)vblk * a.num_kv_heads + kvh];
            }
            const int key0 = kb + 8 * g4;
            float p[8];
            float mx = -INFINITY;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int key = key0 + 4 * t + r;
                    const float v = s[t][r] * sk;
                    p[4 * t + r] = (key < key_end && key < klim) ? v : -INFINITY;
                    mx = fmaxf(mx, p[4 * t + r]);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run, mx);
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2f(m_run - m_use);
            float psum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                p[e] = exp2f(p[e] - m_use);
                psum += p[e];
            }
            l_run = l_run * alpha + psum;
            m_run = m_new;
#pragma unroll
            for (int i = 0; i < NT; ++i) acc[i] *= alpha;

            // e4m3: p times the V scale as a bf16 pair hi + lo (two MFMAs), so
            // that the scale is not rounded to bf16 along with every term
            bf16x8_t pf, pl;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if constexpr (FP8) {
                    const float x = p[e] * sv;
                    pf[e] = (__bf16)x;
                    pl[e] = (__bf16)(x - (float)pf[e]);
                } else {
                    pf[e] = (__bf16)p[e];
                }
            }

            if (kb + 32 > key_end) {  // zero V columns past the end: 0 * NaN is NaN
                const int valid = key_end - key0;
                const uint32_t keep = valid >= 8 ? 0xFFu : (valid <= 0 ? 0u : ((1u << valid) - 1u));
#pragma unroll
                for (int i = 0; i < NT; ++i) vr[i] = kv::mask(vr[i], keep);
            }
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const bf16x8_t vf = kv::widen(vr[i]);
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, acc[i], 0, 0, 0);
                if constexpr (FP8) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pl, acc[i], 0, 0, 0);
            }
        }
    };
    if (shape & kItemShared) sweep(Flag<false>{});
    else sweep(Flag<true>{});

    float l_tot = l_run + __shfl_xor(l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);
    if (!qvalid) return;
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    float *dst;
    if (part < 0) {
        dst = a.out + ((int64_t)tok * a.num_q_heads + head) * D;
    } else {
        dst = a.part_o + (int64_t)(part + c16) * D;
        if (g4 == 0) a.part_lse[part + c16] = l_tot > 0.f ? m_run + log2f(l_tot) : -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) *(f32x4_t *)(dst + 16 * i + 4 * g4) = acc[i] * inv;
}

// `words` 32-bit words by workgroups of 256 threads, 16 bytes per thread and
// step; part of `parts`
__device__ __forceinline__ void copy_words(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst,
                                           int64_t words, int part, int parts) {
    const int64_t n16 = words / 4;
    const int64_t stride = (int64_t)parts * 256;
    for (int64_t i = (int64_t)part * 256 + threadIdx.x; i < n16; i += stride)
        ((u32x4_t *)dst)[i] = ((const u32x4_t *)src)[i];
    const int64_t t = 4 * n16 + threadIdx.x;
    if (part == 0 && t < words) dst[t] = src[t];
}

template <int D, bool FP8>
__global__ __launch_bounds__(256) void attn_kernel(AttnArgs a) {
    if ((int)blockIdx.x >= a.copy_first) {
        copy_words(a.copy_src, a.copy_dst, a.copy_words, blockIdx.x - a.copy_first,
                   gridDim.x - a.copy_first);
        return;
    }
    decode_body<D, FP8>(a, blockIdx.x, threadIdx.x);
}

// ------------------------------------------------------------------ prefill
//
// One workgroup = 8 waves x 32 query vectors (consecutive tokens of one
// prefill chunk x the query heads of one KV head), one workgroup per CU.
// K/V tiles of 64 keys live in a 3-stage LDS ring as bf16 (e4m3 caches: V as
// fp16), shared by the eight waves; bf16 tiles are requested two tiles ahead:
//   K  [64 keys][D]            16-byte chunk q of row r stored at q ^ kswz(r)
//   V  [4 blocks][D/16][2][16][8]  per block and 16 rows d of V^T, keys 0-7
//                              of the 16 rows, then keys 8-15 (16 bytes each)
// kswz maps the key-row bits that differ between the 16 lanes of an MFMA
// operand read onto distinct chunks, so every 16-lane read of 16 bytes per
// lane touches all 64 LDS banks once; a 16-lane V operand read is 256
// contiguous bytes.  (Rows of 32 bytes with the halves swapped on bit 3 of d
// also spread 16 lanes over 64 banks, yet cost 4 bank-conflict cycles per
// read on gfx950, measured with SQ_LDS_BANK_CONFLICT; this layout costs none.)
// bf16 pools are copied global -> LDS directly (global_load_lds_dwordx4, no
// staging registers); e4m3 pools go through registers and are widened on the
// way in: K to bf16, V to fp16 after multiplication by its (block, head) scale
// (K scales multiply the logits instead).  Tiles of keys at or past the last
// token's position get their V entries zeroed (0 * NaN is NaN for unwritten
// slots).

constexpr int kPfKeys = 64;
constexpr int kPfLdsLimit = 160 * 1024;   // LDS of one gfx950 CU

// Workgroup shape: W waves (32 query vectors each) and an S-stage LDS ring.
#ifndef ECHO_PF_WAVES
#define ECHO_PF_WAVES 8
#endif
#ifndef ECHO_PF_STAGES
#define ECHO_PF_STAGES 3
#endif
constexpr int kPfWaves = ECHO_PF_WAVES;
constexpr int kPfThreads = 64 * kPfWaves;
constexpr int kPfStages = ECHO_PF_STAGES;
static_assert(32 * kPfWaves == kPrefillQueries, "prefill tile size");

template <int D>
struct PfLds {
    static constexpr int KBYTES = kPfKeys * 2 * D;   // K region of a stage
    static constexpr int VBYTES = 4 * 16 * D * 2;    // V region of a stage
    static constexpr int STAGE = KBYTES + VBYTES;    // bytes
    static constexpr int BYTES = kPfStages * STAGE + kPfStages * 4 * 4;  // + 4 bytes per block id
};

// s_waitcnt operand: vmcnt(n) with expcnt and lgkmcnt left free
constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
// vmcnt(n) and lgkmcnt(0): also every LDS write of this wave has landed
constexpr int waitcnt_vm_lds(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

typedef __attribute__((address_space(3))) void lds_void_t;

// One prefill descriptor di (a tile's tokens, or a piece of their keys) for
// KV head kvh; all kPfThreads threads of the workgroup take part.
// DENSE (head_dim 64): two workgroups per CU, see prefill_kernel.
template <int D, bool FP8, bool DENSE>
__device__ __forceinline__ void prefill_piece(const PrefillArgs &a, int kvh, int di) {
    typedef KV<FP8> kv;
    typedef typename kv::T KT;
    typedef typename kv::VRaw Raw;   // 8 codes (16 or 8 bytes)
    typedef PfLds<D> LD;
    // P.V operand types.  e4m3: V times its block scale, and P, are fp16 (11
    // significant bits: the scaled values are not bf16-exact, and bf16's 8
    // bits would put errors up to 2^-9 |v| on rows with few keys)
    typedef std::conditional_t<FP8, _Float16, __bf16> PE;
    typedef std::conditional_t<FP8, f16x8_t, bf16x8_t> PT;
    // chunk guard of the lazy rescale (log2 units): probabilities stay below
    // 2^kGuard, inside fp16's range for e4m3
    constexpr float kGuard = FP8 ? 15.f : 64.f;
    constexpr int NC = D / 32, NT = D / 16;
    constexpr int CHUNKS = D / 8;              // 16-byte chunks per K row
    constexpr int NJ = D / (8 * kPfWaves);     // 1 KiB copies per wave per region per tile
    // chunk swizzle of K row r (see above): rows 32ch + 8(c16>>2) + 4t + (c16&3)
    // are read by lane c16, so the swizzle is a function of c16 alone
    auto kswz = [](int r) -> int {
        return D == 128 ? ((r & 3) | ((r >> 1) & 0xC)) : (((r >> 1) & 1) | ((r >> 2) & 6));
    };
    extern __shared__ __align__(16) uint8_t lds[];
    float *lscale = (float *)(lds + kPfStages * LD::STAGE);  // [stage][4]: K scales
    int32_t *lids = (int32_t *)(lscale + kPfStages * 4);      // the row's block ids

    const int32_t *dp = (const int32_t *)(a.pdesc + di);
    const int row = __builtin_amdgcn_readfirstlane(dp[0]);
    const int tok0 = __builtin_amdgcn_readfirstlane(dp[1]);
    const int ntok = __builtin_amdgcn_readfirstlane(dp[2]);
    const int key_end = __builtin_amdgcn_readfirstlane(dp[3]);
    const int key_begin = __builtin_amdgcn_readfirstlane(dp[4]);   // piece of the keys
    const int part = __builtin_amdgcn_readfirstlane(dp[5]);        // >= 0: partial results
    const int kfull = __builtin_amdgcn_readfirstlane(dp[6]);       // keys every token sees

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, c16 = lane & 15;
    const int G = a.group;
    // token t of the row sits at position t - (q_start[row + 1] - seq_lens[row])
    // and sees the keys up to and including it
    const int klim_base = __builtin_amdgcn_readfirstlane(a.seq_lens[row] - a.q_start[row + 1] + 1);

    // this lane's two query columns (N tiles nn = 0, 1)
    bf16x8_t qf[2][NC];
    int klim[2], qtok[2], qhead[2];
    bool qok[2];
#pragma unroll
    for (int nn = 0; nn < 2; ++nn) {
        const int qi = 32 * wave + 16 * nn + c16;
        const int tl = qi / G;
        qok[nn] = tl < ntok;
        qtok[nn] = tok0 + (qok[nn] ? tl : 0);
        qhead[nn] = kvh * G + (qi - tl * G);
        klim[nn] = qok[nn] ? klim_base + qtok[nn] : 0;
        const uint16_t *qp = a.q + ((int64_t)qtok[nn] * a.num_q_heads + qhead[nn]) * D + 8 * g4;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            u32x4_t w = {0u, 0u, 0u, 0u};
            if (qok[nn]) w = *(const u32x4_t *)(qp + 32 * c);
            qf[nn][c] = __builtin_bit_cast(bf16x8_t, w);
        }
    }

    f32x4_t acc[2][NT];
#pragma unroll
    for (int nn = 0; nn < 2; ++nn)
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[nn][i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    float m_run[2] = {-INFINITY, -INFINITY};
    // derived from m_run: the exponent offset (-m_run, 0 while m_run is -inf)
    // and the two lazy-rescale thresholds; kept and refreshed when m_run moves, or
    // for DENSE, whose registers are short, taken from it at each use
    float neg_at[2] = {0.f, 0.f}, hig_at[2] = {-INFINITY, -INFINITY}, hi8_at[2] = {-INFINITY, -INFINITY};
    auto m_neg = [&](int nn) -> float {
        if constexpr (DENSE) return m_run[nn] == -INFINITY ? 0.f : -m_run[nn];
        else return neg_at[nn];
    };
    auto m_hig = [&](int nn) -> float { return DENSE ? m_run[nn] + kGuard : hig_at[nn]; };
    auto m_hi8 = [&](int nn) -> float { return DENSE ? m_run[nn] + 8.f : hi8_at[nn]; };
    // The softmax denominator is a P.V product with V = 1 (every row of
    // lacc[nn] holds the column sum), so it sums exactly the rounded weights
    // that P.V uses and costs one MFMA per chunk instead of 16 adds per lane
    // (e4m3 V carries its block scale in the widened values, so the weights
    // are plain probabilities there too).
    f32x4_t lacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    PT ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (PE)1.0f;

    const int32_t *btr = a.block_tables + (int64_t)row * a.max_blocks_per_row;
    const int64_t blk_stride = (int64_t)a.num_kv_heads * 16 * D;
    const KT *kbase = (const KT *)a.k + (int64_t)kvh * 16 * D;
    const KT *vbase = (const KT *)a.v + (int64_t)kvh * 16 * D;
    const int ntiles = (key_end + kPfKeys - 1) / kPfKeys;   // tiles kt0 .. ntiles-1 of the row
    const int kt0 = key_begin / kPfKeys;
    const int kb0 = key_begin / 16, nblk = (key_end + 15) / 16 - kb0;   // blocks staged
    // keys every query of the workgroup sees: tiles below this need no mask

    // The row's block ids (up to the last key of the tile) are staged in LDS
    // once; tile block indices past the last block are clamped so that every
    // copy is unconditional (keys past key_end are zeroed or masked instead).
    for (int e = tid; e < nblk; e += kPfThreads) lids[e] = btr[kb0 + e];
    __syncthreads();
    auto blk_of = [&](int kt, int b) -> int { return lids[min(4 * (kt - kt0) + b, nblk - 1)]; };

    // This wave's NJ copies of a tile all fall in block `bsel` of the tile's
    // four; per lane, where each 16-byte piece comes from inside the block is
    // the same for every tile, so only the block id (read from LDS once per
    // tile, a step ahead, and made scalar) changes.
    static_assert((32 * D) % (NJ * 1024) == 0, "a wave's copies stay inside one block");
    const int bsel = wave * NJ * 1024 / (32 * D);
    // (unsigned for DENSE: a scalar base and a 32-bit offset, fewer registers)
    std::conditional_t<DENSE, uint32_t, int> k_off[NJ], v_off[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int off = (wave * NJ + j) * 1024 + 16 * lane;   // byte offset in the K / V region
        const int r = off / (2 * D), q = ((off / 16) % CHUNKS) ^ kswz(r);
        k_off[j] = (r & 15) * D + 8 * q;
        // V: 16-byte unit u of the block's region holds keys 8h..8h+7 of row
        // d = 16(u / 32) + u % 16, h = (u / 16) % 2
        const int u = (off % (32 * D)) / 16;
        const int d = 16 * (u >> 5) + (u & 15), h = (u >> 4) & 1;
        v_off[j] = d * 16 + 8 * h;
    }
    auto tile_id = [&](int kt) -> int { return lids[min(4 * (kt - kt0) + bsel, nblk - 1)]; };

    Raw kreg[FP8 ? NJ : 1], vreg[FP8 ? NJ : 1];
    float sreg = 0.f, vscale = 1.f;
    auto issue_tile = [&](int kt, int buf, int id) {
        uint8_t *kl = lds + buf * LD::STAGE;
        uint8_t *vl = kl + LD::KBYTES;
        const int blk = __builtin_amdgcn_readfirstlane(id);
        const KT *kb = kbase + (int64_t)blk * blk_stride;
        const KT *vb = vbase + (int64_t)blk * blk_stride;
        if constexpr (!FP8) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                __builtin_amdgcn_global_load_lds((const void *)(kb + k_off[j]),
                                                 (lds_void_t *)(kl + (wave * NJ + j) * 1024), 16, 0, 0);
                __builtin_amdgcn_global_load_lds((const void *)(vb + v_off[j]),
                                                 (lds_void_t *)(vl + (wave * NJ + j) * 1024), 16, 0, 0);
            }
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                kreg[j] = pool_load<false, Raw>(kb + k_off[j]);
                vreg[j] = pool_load<false, Raw>(vb + v_off[j]);
            }
            // the V scale of this wave's block goes into the widened values;
            // the K scales of the tile's four blocks scale the logits
            vscale = a.v_scale[(int64_t)blk * a.num_kv_heads + kvh];
            if (tid < 4) sreg = a.k_scale[(int64_t)blk_of(kt, tid) * a.num_kv_heads + kvh];
        }
    };
    // e4m3 only: widen the staged registers into LDS, V times its block's
    // scale as fp16
    auto store_tile = [&](int buf) {
        if constexpr (FP8) {
            uint8_t *kl = lds + buf * LD::STAGE;
            uint8_t *vl = kl + LD::KBYTES;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                *(u32x4_t *)(kl + (wave * NJ + j) * 1024 + 16 * lane) =
                    __builtin_bit_cast(u32x4_t, kv::widen(kreg[j]));
                const bf16x8_t w = kv::widen(vreg[j]);
                PT v;
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (PE)((float)w[e] * vscale);
                *(u32x4_t *)(vl + (wave * NJ + j) * 1024 + 16 * lane) = __builtin_bit_cast(u32x4_t, v);
            }
            if (tid < 4) lscale[buf * 4 + tid] = sreg;
        }
    };
    // zero V of keys at or past key_end in the tile of buffer `buf`
    auto zero_tail = [&](int kt, int buf) {
        uint16_t *vl = (uint16_t *)(lds + buf * LD::STAGE + LD::KBYTES);
        for (int e = tid; e < 4 * D * 2; e += kPfThreads) {  // 16-byte units of the four blocks
            const int b = e / (2 * D), u = e % (2 * D);
            const int key = kPfKeys * kt + 16 * b + 8 * ((u >> 4) & 1);
            uint16_t *dst = vl + b * 16 * D + 8 * u;
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (key + x >= key_end) dst[x] = 0;
        }
    };

    const float scale = a.scale_log2;
    const int ksel_row = 8 * (c16 >> 2) + (c16 & 3);  // + 4t + 32ch: S^T row -> key
    const int kswz_lane = kswz(ksel_row);

    // One 64-key tile in LDS buffer `buf`, as a two-chunk software pipeline:
    //   QK(c0) | QK(c1) + exp(c0) | PV(c0) + exp(c1) | PV(c1)
    // so that each run of MFMAs has independent VALU work to co-issue with.
    // Probabilities are taken against a reference m_run (log2 units) fixed
    // for the tile; it moves at the end of the tile when the tile's max
    // exceeds it by more than 8 (rescaling acc and l), or, before a chunk's
    // exponentials, when a chunk's max exceeds it by more than kGuard (rare
    // guard that also covers the first tile, where m_run is still -inf).
    // Both tests take any lane whose own scores cross the threshold, which is
    // the same as the column's maximum crossing it.
    auto qk = [&](const uint8_t *kl, int ch, f32x4_t (&sc)[2][2]) {
        // scheduling hint for the MFMA runs of a region (LLVM's IGroupLP mode 1,
        // single-wave small-GEMM interleave): 2-3% faster on long prefills
        __builtin_amdgcn_iglp_opt(1);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            sc[t][0] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
            sc[t][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint8_t *krow = kl + (32 * ch + ksel_row + 4 * t) * (2 * D);
                const bf16x8_t kf = *(const bf16x8_t *)(krow + 16 * ((4 * c + g4) ^ kswz_lane));
#pragma unroll
                for (int nn = 0; nn < 2; ++nn)
                    sc[t][nn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[nn][c], sc[t][nn], 0, 0, 0);
            }
    };
    // mask, and this lane's max over its 8 raw scores of each query column in
    // log2 units (the column's max over its 4 lanes is formed only on the rare
    // rescale path); f receives the chunk's raw score -> log2 factor, which for
    // e4m3 includes the K scale of this lane's block (positive, so the max of
    // the raw scores gives the max of the scaled ones)
    auto prep = [&](int buf, int kt, int ch, bool masked, f32x4_t (&sc)[2][2], float (&mc)[2], float &f) {
        f = scale;
        if constexpr (FP8) f = scale * lscale[buf * 4 + 2 * ch + (g4 >> 1)];
        const int key0 = kPfKeys * kt + 32 * ch + 8 * g4;
#pragma unroll
        for (int nn = 0; nn < 2; ++nn) {
            float mx = -INFINITY;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v = sc[t][nn][r];
                    if (masked) v = (key0 + 4 * t + r < klim[nn]) ? v : -INFINITY;
                    sc[t][nn][r] = v;
                    mx = fmaxf(mx, v);
                }
            mc[nn] = mx * f;
        }
    };
    auto rescale = [&](const float (&mnew)[2]) {
#pragma unroll
        for (int nn = 0; nn < 2; ++nn) {
            const float alpha = m_run[nn] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run[nn] - mnew[nn]);
            lacc[nn] *= alpha;
#pragma unroll
            for (int i = 0; i < NT; ++i) acc[nn][i] *= alpha;
            m_run[nn] = mnew[nn];
            if constexpr (!DENSE) {
                neg_at[nn] = mnew[nn] == -INFINITY ? 0.f : -mnew[nn];
                hig_at[nn] = mnew[nn] + kGuard;
                hi8_at[nn] = mnew[nn] + 8.f;
            }
        }
    };
    // exponentials of one chunk against m_run, packed to bf16 (fp16 for e4m3)
    auto expo = [&](const f32x4_t (&sc)[2][2], PT (&pf)[2], float f) {
#pragma unroll
        for (int nn = 0; nn < 2; ++nn) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float pe = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[t][nn][r], f, m_neg(nn)));
                    pf[nn][4 * t + r] = (PE)pe;
                }
        }
    };
    auto pv = [&](const uint8_t *vl, int ch, const PT (&pf)[2]) {
        __builtin_amdgcn_iglp_opt(1);   // as in qk
        const uint8_t *vrow = vl + (2 * ch + (g4 >> 1)) * (32 * D) + (g4 & 1) * 256 + c16 * 16;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const PT vf = *(const PT *)(vrow + i * 16 * 32);
#pragma unroll
            for (int nn = 0; nn < 2; ++nn) acc[nn][i] = mfma_pv(vf, pf[nn], acc[nn][i]);
        }
#pragma unroll
        for (int nn = 0; nn < 2; ++nn)
            lacc[nn] = mfma_pv(ones, pf[nn], lacc[nn]);
    };
    auto tile_piped = [&](int buf, int kt, bool masked) {
        const uint8_t *kl = lds + buf * LD::STAGE;
        const uint8_t *vl = kl + LD::KBYTES;
        f32x4_t s0[2][2], s1[2][2];
        float m0[2], m1[2], f0, f1;
        PT p0[2], p1[2];
        qk(kl, 0, s0);
        prep(buf, kt, 0, masked, s0, m0, f0);
        if (__any(m0[0] > m_hig(0) || m0[1] > m_hig(1))) {
            const float mn[2] = {fmaxf(m_run[0], wave_max_xor16_32(m0[0])),
                                 fmaxf(m_run[1], wave_max_xor16_32(m0[1]))};
            rescale(mn);
        }
        qk(kl, 1, s1);          // MFMA ...
        expo(s0, p0, f0);       // ... with the exponentials of chunk 0
        prep(buf, kt, 1, masked, s1, m1, f1);
        if (__any(m1[0] > m_hig(0) || m1[1] > m_hig(1))) {
            // chunk 0's probabilities, not yet added, move with the reference
            const float mn[2] = {fmaxf(m_run[0], wave_max_xor16_32(m1[0])),
                                 fmaxf(m_run[1], wave_max_xor16_32(m1[1]))};
#pragma unroll
            for (int nn = 0; nn < 2; ++nn) {
                const float alpha =
                    m_run[nn] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run[nn] - mn[nn]);
#pragma unroll
                for (int e = 0; e < 8; ++e) p0[nn][e] = (PE)((float)p0[nn][e] * alpha);
            }
            rescale(mn);
        }
        pv(vl, 0, p0);          // MFMA ...
        expo(s1, p1, f1);       // ... with the exponentials of chunk 1
        pv(vl, 1, p1);
        const float mt[2] = {vmax(m0[0], m1[0]), vmax(m0[1], m1[1])};
        if (__any(mt[0] > m_hi8(0) || mt[1] > m_hi8(1))) {
            const float mc[2] = {wave_max_xor16_32(mt[0]), wave_max_xor16_32(mt[1])};
            const float mn[2] = {mc[0] > m_hi8(0) ? mc[0] : m_run[0],
                                 mc[1] > m_hi8(1) ? mc[1] : m_run[1]};
            rescale(mn);
        }
    };

    // The same tile a chunk at a time, for DENSE: half the live scores and
    // probabilities, and the other workgroup's waves to co-issue with.
    auto tile_serial = [&](int buf, int kt, bool masked) {
        const uint8_t *kl = lds + buf * LD::STAGE;
        const uint8_t *vl = kl + LD::KBYTES;
        float mt[2] = {-INFINITY, -INFINITY};
#pragma unroll
        for (int ch = 0; ch < 2; ++ch) {
            f32x4_t sc[2][2];
            float m[2], f;
            PT pr[2];
            qk(kl, ch, sc);
            prep(buf, kt, ch, masked, sc, m, f);
            if (__any(m[0] > m_hig(0) || m[1] > m_hig(1))) {
                const float mn[2] = {fmaxf(m_run[0], wave_max_xor16_32(m[0])),
                                     fmaxf(m_run[1], wave_max_xor16_32(m[1]))};
                rescale(mn);
            }
            expo(sc, pr, f);
            pv(vl, ch, pr);
            mt[0] = vmax(mt[0], m[0]);
            mt[1] = vmax(mt[1], m[1]);
        }
        if (__any(mt[0] > m_hi8(0) || mt[1] > m_hi8(1))) {
            const float mc[2] = {wave_max_xor16_32(mt[0]), wave_max_xor16_32(mt[1])};
            const float mn[2] = {mc[0] > m_hi8(0) ? mc[0] : m_run[0],
                                 mc[1] > m_hi8(1) ? mc[1] : m_run[1]};
            rescale(mn);
        }
    };
    auto tile = [&](int buf, int kt, bool masked) {
        if constexpr (DENSE) tile_serial(buf, kt, masked);
        else tile_piped(buf, kt, masked);
    };

    // Pipeline.  bf16: iteration kt loads the block ids of tile kt+3, starts
    // the copies of tile kt+2, computes tile kt, then waits until its own
    // copies of tile kt+1 have landed (the newer ones stay in flight) and
    // meets the other waves at the barrier.  e4m3: tile kt+1 is staged in
    // registers during tile kt and widened into LDS before the barrier.
    constexpr int LA = (FP8 || kPfStages == 2) ? 1 : 2;  // tiles in flight ahead
    const int tail_tile = (kPfKeys * ntiles > key_end) ? ntiles - 1 : -1;
    // LDS buffer of tile kt: (kt - kt0) % kPfStages
    issue_tile(kt0, 0, tile_id(kt0));
    store_tile(0);
    if (LA == 2 && ntiles > kt0 + 1) issue_tile(kt0 + 1, 1, tile_id(kt0 + 1));
    int id_ahead = tile_id(kt0 + LA);   // block id of the next tile to issue
    // (e4m3 tiles reach LDS through ds_write, which the barrier does not wait
    // for: this wave's writes must have landed before others read them)
    if (LA == 2 && ntiles > kt0 + 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * NJ));
    else __builtin_amdgcn_s_waitcnt(FP8 ? waitcnt_vm_lds(0) : waitcnt_vm(0));
    __builtin_amdgcn_s_barrier();
    if (tail_tile == kt0) {
        zero_tail(kt0, 0);
        __syncthreads();
    }

    auto step = [&](int kt, bool masked) {
        const int buf = (kt - kt0) % kPfStages;
        bool ahead = false;   // copies of tile kt+2 issued after those of kt+1
        if (kt + LA < ntiles) {
            issue_tile(kt + LA, (kt + LA - kt0) % kPfStages, id_ahead);
            ahead = LA == 2;
        }
        id_ahead = tile_id(kt + LA + 1);
        tile(buf, kt, masked);
        if (kt + 1 < ntiles) {
            if constexpr (LA == 1) store_tile((kt + 1 - kt0) % kPfStages);
            if (ahead) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * NJ));
            else __builtin_amdgcn_s_waitcnt(FP8 ? waitcnt_vm_lds(0) : waitcnt_vm(0));
            __builtin_amdgcn_s_barrier();
            if (kt + 1 == tail_tile) {
                zero_tail(kt + 1, (kt + 1 - kt0) % kPfStages);
                __syncthreads();
            }
        }
    };
    // tiles every query sees in full, then the diagonal tiles with the mask
    const int nfull = min(kfull / kPfKeys, ntiles);
    for (int kt = kt0; kt < nfull; ++kt) step(kt, false);
    for (int kt = max(nfull, kt0); kt < ntiles; ++kt) step(kt, true);

    // DENSE takes the query columns again, from an index the compiler cannot
    // see through: kept from the prologue they hold registers through the loop
    int q0 = 32 * wave + c16;
    if constexpr (DENSE) asm("" : "+v"(q0));
#pragma unroll
    for (int nn = 0; nn < 2; ++nn) {
        const float l_tot = lacc[nn][0];
        if constexpr (DENSE) {
            const int qi = q0 + 16 * nn, tl = qi / G;
            if (tl >= ntok) continue;
            qtok[nn] = tok0 + tl;
            qhead[nn] = kvh * G + (qi - tl * G);
        } else if (!qok[nn]) {
            continue;
        }
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        float *dst;
        if (part < 0) {
            dst = a.out + ((int64_t)qtok[nn] * a.num_q_heads + qhead[nn]) * D + 4 * g4;
        } else {
            // the slot the merge kernel reads for (token, head) of this piece:
            // part + (kvh * head_chunks + hc) * ntok * heads_per_chunk + token * nh + jh
            const int qi = q0 + 16 * nn, tl = qi / G, hg = qi - tl * G;
            const int hc = hg / 16, jh = hg - 16 * hc;
            const int nh = min(a.heads_per_chunk, G - 16 * hc);
            const int64_t slot = part + (int64_t)(kvh * a.head_chunks + hc) * ntok * a.heads_per_chunk +
                                 (int64_t)tl * nh + jh;
            dst = a.part_o + slot * D + 4 * g4;
            if (g4 == 0) a.part_lse[slot] = l_tot > 0.f ? m_run[nn] + log2f(l_tot) : -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < NT; ++i) *(f32x4_t *)(dst + 16 * i) = acc[nn][i] * inv;
    }
}

// One prefill workgroup: P is its physical workgroup index in the prefill
// grid (8 * per_xcd workgroups).  Its descriptor may name a second one
// (a piece of another tile's keys) that the workgroup runs next.
template <int D, bool FP8, bool DENSE>
__device__ __forceinline__ void prefill_body(const PrefillArgs &a, int P) {
    const int L = (P % 8) * a.per_xcd + P / 8;  // consecutive logical tiles share an XCD
    if (L >= a.n_logical) return;
    const int kvh = L / a.n_pdesc;
    int di = L - kvh * a.n_pdesc;
    if (a.counts && di >= ro_load(a.counts, kHdrPdesc)) return;
    for (;;) {
        prefill_piece<D, FP8, DENSE>(a, kvh, di);
        if constexpr (DENSE) break;   // no chains there, and their loop costs registers
        const int next = __builtin_amdgcn_readfirstlane(((const int32_t *)(a.pdesc + di))[7]);
        if (next <= 0) break;
        __syncthreads();   // the next descriptor refills the LDS ring and block ids
        di = next - 1;
    }
}

// One workgroup per CU at head_dim 128 (232 VGPRs, e4m3 246).  At head_dim 64
// half the products meet the same softmax work, and the waves of one workgroup,
// which a barrier per tile keeps in step, leave the matrix cores idle; DENSE holds
// a wave to 128 VGPRs, without spilling, so that two workgroups share a CU, and
// overlaps one workgroup's softmax with the other's products instead of pipelining
// the two chunks of a tile.  Chained descriptors, which only launches of at most
// one round have, are left to the other form: the loop over them holds addresses
// in registers.  12 prompts of 84-1,428 tokens (GQA 64/8), the whole call: 157 ->
// 131 us, e4m3 171 -> 138 (with 6 and 15 registers spilled 138 and 152); the
// kernel, averaged under a trace, 138 and 148 us.
template <int D, bool FP8, bool DENSE>
__global__ __launch_bounds__(kPfThreads, DENSE ? 4 : 1) void prefill_kernel(PrefillArgs a) {
    prefill_body<D, FP8, DENSE>(a, blockIdx.x);
}

// -------------------------------------------------------------------- merge
//
// Lanes in four 16-lane groups, each lane owning D/16 consecutive elements of a
// head's output row.  A group takes its entries 16 at a time (one per lane:
// slot and lse loaded in parallel), rescales its running sums to the new
// maximum, then adds the entries' partial rows, four independent loads at a
// time.  Bound by that chain of loads (entries -> lse -> rows, four deep for 16
// entries) until the partial rows fill the memory's time, so a wave takes
//   WIDE   one head of a token, every group a quarter of its entries, combined
//          at the end: the shortest chain, for rows of many entries and for
//          merges that leave the chip idle
//   else   four heads of a token, a head per group: the fewest waves
// (Eight loads at a time instead of four: 0.5-1 us slower, two waves per SIMD
// fewer.)  8 decode rows of up to 64 entries: 7.0 -> 4.7 us; one row of 64
// entries: 12.6 -> 6.7 us; 32 rows of up to 34 beside 320 tokens of two: 11.5 ->
// 6.7 us.

template <int D, bool WIDE>
__device__ __forceinline__ void merge_heads(const MergeArgs &a, int row, int h, int lane) {
    constexpr int PER = D / 16;   // floats per lane
    constexpr int NV = PER / 4;   // 16-byte loads per lane and partial row
    constexpr int BATCH = 4;
    constexpr int GROUPS = WIDE ? 4 : 1;   // groups that share the entries
    const int c16 = lane & 15, base = lane & 48;
    const int g = WIDE ? lane >> 4 : 0;
    const bool hok = h < a.num_q_heads;
    const int tok = a.merge_tok[row];
    const int e0 = a.merge_ptr[row], e1 = a.merge_ptr[row + 1];
    // where head h of a slice's query i lands inside a descriptor's slots
    const int kvh = h / a.group;
    const int hc = (h - kvh * a.group) / 16;
    const int jh = h - kvh * a.group - hc * 16;
    const int nh = min(a.heads_per_chunk, a.group - hc * 16);
    const int rem = kvh * a.head_chunks + hc;
    f32x4_t acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, wsum = 0.f;
    // every lane stays in the loop: the lane exchanges read all of them
    for (int eb = e0; eb < e1; eb += 16 * GROUPS) {
        const int e = eb + GROUPS * c16 + g;
        int slot = 0;
        float lse = -INFINITY;
        if (hok && e < e1) {
            const int part = a.merge_ent[2 * e], sh = a.merge_ent[2 * e + 1];
            slot = part + rem * (sh & 0x3FF) * a.heads_per_chunk + (sh >> 10) * nh + jh;
            lse = a.part_lse[slot];
        }
        float bm = lse;
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) bm = fmaxf(bm, __shfl_xor(bm, off));
        const float m_new = fmaxf(mx, bm);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = exp2f(mx - m_use);   // 0 while mx is -inf
        const float w = lse == -INFINITY ? 0.f : exp2f(lse - m_use);
        float ws = w;
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) ws += __shfl_xor(ws, off);
        wsum = wsum * alpha + ws;
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[k] *= alpha;
        mx = m_new;
        const int most = min(16, (e1 - eb + GROUPS - 1) / GROUPS);   // entries of group 0
        const int n = WIDE ? min(16, (e1 - eb - g + 3) >> 2) : most; // of this group
        auto load = [&](int i, f32x4_t (&v)[NV], float &wi) {
            const int si = __shfl(slot, base + i);
            wi = __shfl(w, base + i);
            const f32x4_t *po = (const f32x4_t *)(a.part_o + (int64_t)si * D + c16 * PER);
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                if constexpr (WIDE) {
                    v[k] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
                    if (i < n) v[k] = po[k];
                } else {
                    v[k] = po[k];
                }
            }
        };
        int i = 0;
        for (; WIDE ? i < most : i + BATCH <= most; i += BATCH) {
            f32x4_t v[BATCH][NV];
            float wi[BATCH];
#pragma unroll
            for (int j = 0; j < BATCH; ++j) load((i + j) & 15, v[j], wi[j]);
#pragma unroll
            for (int j = 0; j < BATCH; ++j)
#pragma unroll
                for (int k = 0; k < NV; ++k) acc[k] += (!WIDE || i + j < n ? wi[j] : 0.f) * v[j][k];
        }
        if constexpr (!WIDE)
            for (; i < most; ++i) {
                f32x4_t v[NV];
                float wi;
                load(i, v, wi);
#pragma unroll
                for (int k = 0; k < NV; ++k) acc[k] += wi * v[k];
            }
    }
    if constexpr (WIDE) {
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float om = __shfl_xor(mx, off);
            const float m_new = fmaxf(mx, om);
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2f(mx - m_use), beta = exp2f(om - m_use);
            wsum = wsum * alpha + __shfl_xor(wsum, off) * beta;
#pragma unroll
            for (int k = 0; k < NV; ++k)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    acc[k][x] = acc[k][x] * alpha + __shfl_xor(acc[k][x], off) * beta;
            mx = m_new;
        }
        if (g) return;
    }
    if (!hok) return;
    const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
    f32x4_t *o = (f32x4_t *)(a.out + ((int64_t)tok * a.num_q_heads + h) * D + c16 * PER);
#pragma unroll
    for (int k = 0; k < NV; ++k) o[k] = acc[k] * inv;
}

// The first a.n_wide rows go a head per wave, the others four.
template <int D>
__global__ __launch_bounds__(256) void merge_kernel(MergeArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t m = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (m >= a.n_waves) return;
    const int64_t wide = a.n_wide * a.num_q_heads;
    const int per = m < wide ? a.num_q_heads : (a.num_q_heads + 3) / 4;
    const int64_t x = m < wide ? m : m - wide;
    const int64_t r = x >> 32 ? x / per : (int64_t)((uint32_t)x / (uint32_t)per);
    const int k = (int)(x - r * per), row = (int)(m < wide ? r : r + a.n_wide);
    if (a.counts && row >= ro_load(a.counts, kHdrMergeRows)) return;
    if (m < wide) merge_heads<D, true>(a, row, k, lane);
    else merge_heads<D, false>(a, row, 4 * k + (lane >> 4), lane);
}

// ------------------------------------------------------- device-built plan
//
// For batches given without host mirrors: the plan is built on the GPU from
// the row metadata, with no prefix grouping.  A row is checked (its metadata
// and block ids) before it gets work; rows whose metadata is inconsistent, or
// whose tiles would not fit the prefill region (which only an inconsistent
// q_start can cause), get none and are counted in the header, so every kernel
// after the plan stays inside its buffers.  A row of one new token is decode
// work whatever its kind: the same sum, without a prefill workgroup for it.
//
// What bounds it is latency: a handful of dependent loads, a scan and the
// stores, for a few hundred descriptors.  So one workgroup does all of it when
// it can check every block id in a few loads per thread, and the descriptors
// are written flat, one per thread whatever row they belong to.  64 rows of up
// to 4,096 keys: 9.6 us, where a check kernel and a thread per row that walked
// its own pieces took 3.6 + 45 us beside 106 us of attention.

__device__ __forceinline__ bool dev_row_ok(const DevPlanArgs &a, int t0, int t1, int L, int kind) {
    const int q = t1 - t0;
    return q >= 1 && L >= q && L <= a.max_seq_len && t0 >= 0 && t1 <= a.num_tokens &&
           (kind == 0 ? q == 1 : kind == 1) && (kind == 0 || L <= a.prefill_max_keys);
}

// One workgroup per row: row_info[r] = 0, or -1 when the row is inconsistent.
__global__ __launch_bounds__(256) void dev_rows_kernel(DevPlanArgs a) {
    const int r = blockIdx.x;
    const int L = a.seq_lens[r];
    const bool ok = dev_row_ok(a, a.q_start[r], a.q_start[r + 1], L, a.row_kind[r]);
    const int nb = ok ? (L + 15) / 16 : 0;
    const int32_t *bt = a.block_tables + (int64_t)r * a.max_blocks_per_row;
    int bad = 0;
    for (int j = threadIdx.x; j < nb; j += 256) {
        const int id = bt[j];
        bad |= (id < 0 || id >= a.num_blocks);
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) a.row_info[r] = ok && !bad ? 0 : -1;
}

constexpr int kPlanThreads = 1024;   // rows per window of dev_plan_kernel
constexpr int kPlanWaves = kPlanThreads / 64;

// What a row adds to the plan: decode pieces, merged rows, merge entries,
// prefill tiles.
struct PlanCount {
    int32_t dec, rows, ent;
    int64_t pf;
};

// Exclusive scan of v over the workgroup's threads, of which only the first
// `live` waves hold anything; tot receives the sum.
__device__ __forceinline__ PlanCount plan_scan(const PlanCount &v, int live, PlanCount *wsum,
                                               PlanCount &tot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    PlanCount inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t d = __shfl_up(inc.dec, off), r = __shfl_up(inc.rows, off),
                      e = __shfl_up(inc.ent, off);
        const int64_t p = __shfl_up(inc.pf, off);
        if (lane >= off) {
            inc.dec += d;
            inc.rows += r;
            inc.ent += e;
            inc.pf += p;
        }
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    PlanCount out = {inc.dec - v.dec, inc.rows - v.rows, inc.ent - v.ent, inc.pf - v.pf};
    tot = {0, 0, 0, 0};
    for (int w = 0; w < live; ++w) {
        const PlanCount x = wsum[w];
        if (w < wave) {
            out.dec += x.dec;
            out.rows += x.rows;
            out.ent += x.ent;
            out.pf += x.pf;
        }
        tot.dec += x.dec;
        tot.rows += x.rows;
        tot.ent += x.ent;
        tot.pf += x.pf;
    }
    return out;
}

// last i in [0, n) with off[i] <= x (off ascending, off[0] <= x)
__device__ __forceinline__ int plan_find(const int32_t *off, int n, int x) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// CHECK: a launch of one workgroup that checks the block ids as well (at most
// kPlanThreads rows); otherwise dev_rows_kernel has, every workgroup scans all
// rows, and the workgroups share the writing.
template <bool CHECK>
__global__ __launch_bounds__(kPlanThreads) void dev_plan_kernel(DevPlanArgs a) {
    __shared__ int32_t row_dec[kPlanThreads], row_pf[kPlanThreads];      // first descriptor
    __shared__ int32_t row_np[kPlanThreads], row_ent[kPlanThreads];      // pieces, first entry
    __shared__ int32_t row_len[kPlanThreads], row_t0[kPlanThreads], row_q[kPlanThreads];
    __shared__ PlanCount wsum[kPlanWaves];
    __shared__ int64_t wsum_l[kPlanWaves];
    __shared__ int32_t pieces[kPlanWaves][64];
    __shared__ int bad_rows, used_pf;
    const int tid = threadIdx.x;
    const int B = a.num_rows;
    if (tid == 0) bad_rows = used_pf = 0;

    int t0 = 0, q = 0, L = 0;
    bool ok = false;
    auto load_row = [&](int r) {
        t0 = q = L = 0;
        ok = false;
        if (r >= B) return;
        t0 = a.q_start[r];
        const int t1 = a.q_start[r + 1];
        L = a.seq_lens[r];
        ok = CHECK ? dev_row_ok(a, t0, t1, L, a.row_kind[r]) : a.row_info[r] == 0;
        q = t1 - t0;
    };
    if constexpr (CHECK) {
        // every (row, block) of the table's used width, eight loads in flight,
        // the first ones beside the row metadata (entries past a row's end are
        // read and not looked at)
        constexpr int N = 8;
        const int W = (a.max_seq_len + 15) / 16;
        const int n = B * W;
        const int dr = kPlanThreads / W, dj = kPlanThreads - dr * W;
        int row = tid / W, j = tid - row * W;   // of the next entry to load
        int id[N], er[N], ej[N];
        auto load = [&](int base) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                er[k] = row;
                ej[k] = base + k * kPlanThreads + tid < n ? j : W;
                id[k] = ej[k] < W ? a.block_tables[(int64_t)row * a.max_blocks_per_row + j] : 0;
                row += dr;
                j += dj;
                if (j >= W) {
                    j -= W;
                    ++row;
                }
            }
        };
        load(0);
        load_row(tid);
        row_np[tid] = ok ? (L + 15) / 16 : 0;
        row_ent[tid] = 0;   // set by a bad block id
        __syncthreads();
        for (int base = 0; base < n; base += N * kPlanThreads) {
            if (base > 0) load(base);
#pragma unroll
            for (int k = 0; k < N; ++k)
                if ((uint32_t)id[k] >= (uint32_t)a.num_blocks && ej[k] < W && ej[k] < row_np[er[k]])
                    row_ent[er[k]] = 1;
        }
        __syncthreads();
        ok = ok && !row_ent[tid];
        __syncthreads();
    }

    // Pieces of decode rows: the host planner's rule (build_plan) on the blocks
    // there are, but no shorter than the descriptor region allows.  The region
    // holds every row cut into pieces of split_blocks, the rule's value for
    // the longest lengths the scalars allow.  (The merge is launched in any case,
    // so the rule's price of a merge has no place here.)
    auto dec_blocks = [&]() -> int { return ok && q == 1 ? (L + 15) / 16 : 0; };
    int64_t blocks = 0;
    {
        int64_t mine = 0;
        for (int base = 0; base < B; base += kPlanThreads) {
            if constexpr (!CHECK) load_row(base + tid);
            mine += dec_blocks();
        }
        row_np[tid] = (int32_t)mine;   // a row's own blocks when one window holds them all
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mine += __shfl_xor(mine, off);
        if ((tid & 63) == 0) wsum_l[tid >> 6] = mine;
        __syncthreads();
        for (int w = 0; w < kPlanWaves; ++w) blocks += wsum_l[w];
    }
    const int64_t units_cap = min<int64_t>(blocks * a.waves_per_desc / kSplitTargetUnits,
                                           a.max_split_blocks);
    const uint32_t room = (uint32_t)(a.cap_desc - B);   // 0: the region holds one piece per row
    int lo = a.split_blocks;                            // shortest piece that fits the region
    if (room > 0 && blocks < ((int64_t)1 << 31))
        lo = min(lo, max(a.min_split_blocks, (int)(((uint32_t)blocks + room - 1) / room)));
    int split = min(a.split_blocks, max(max(lo, kMinSplitBlocks), (int)units_cap));
    if (B <= kPlanThreads) {
        // Waves of the launch for 64 piece lengths from lo to the longest, one
        // per lane (the waves take the rows in turn); then, as the host planner
        // does, the shortest length for each number of workgroups per CU, and
        // the cheapest of those.
        const int longest = max(max(split, (int)units_cap), a.max_split_blocks / kOneGenerationStretch);
        const int step = (longest - lo + 63) / 63;
        const int lane = tid & 63, cand = min(lo + lane * step, longest);
        // pieces of a row by a reciprocal (halfway between the quotients'
        // steps: exact below 2^18 blocks, and near enough above)
        const float inv = 1.0f / (float)cand, half = (float)cand - 0.5f;
        int mine = 0;
        for (int r = tid >> 6; r < B; r += kPlanWaves) mine += (int)(((float)row_np[r] + half) * inv);
        pieces[tid >> 6][lane] = mine;
        __syncthreads();
        int64_t n = 0;
#pragma unroll
        for (int w = 0; w < kPlanWaves; ++w) n += pieces[w][lane];
        n *= a.waves_per_desc;
        int best = 0x7fffffff;
        if (__ballot(n <= a.wave_slots)) {   // (the counts fall with the length)
#pragma unroll
            for (int per_cu = 1; per_cu <= kDecodeWavesPerCu / kWavesPerGroup; ++per_cu) {
                const uint64_t fit = __ballot(n <= a.wave_slots / kDecodeWavesPerCu * (per_cu * kWavesPerGroup));
                if (!fit) continue;
                const int len = min(lo + (__ffsll((unsigned long long)fit) - 1) * step, longest);
                const int cost = decode_cost(per_cu, len, a.light_steps != 0);
                if (10 * (int64_t)cost < 9 * (int64_t)best) {
                    best = cost;
                    split = len;
                }
            }
        }
    }

    int32_t done_dec = 0, done_rows = 0, done_ent = 0;
    int64_t done_pf = 0;
    for (int base = 0; base < B; base += kPlanThreads) {
        const int nr = min(kPlanThreads, B - base);
        const int live = (nr + 63) / 64;
        if constexpr (!CHECK) load_row(base + tid);
        const int nb = dec_blocks();
        const int np = (nb + split - 1) / split;
        const int tiles = ok && q > 1 ? (q + a.tile_tokens - 1) / a.tile_tokens : 0;
        const bool merged = np > 1;
        PlanCount tot;
        const PlanCount at = plan_scan({np, merged ? 1 : 0, merged ? np : 0, tiles}, live, wsum, tot);
        const bool fits = tiles == 0 || done_pf + at.pf + tiles <= a.cap_pdesc;
        row_dec[tid] = at.dec;
        row_pf[tid] = (int32_t)min<int64_t>(at.pf, a.cap_pdesc - min<int64_t>(done_pf, a.cap_pdesc));
        row_np[tid] = np;
        row_ent[tid] = merged ? done_ent + at.ent : -1;
        row_len[tid] = L;
        row_t0[tid] = t0;
        row_q[tid] = q;
        if (base + tid < B && (!ok || !fits)) atomicAdd(&bad_rows, 1);
        if (tiles > 0 && fits) atomicMax(&used_pf, (int)(done_pf + at.pf + tiles));
        if (merged && blockIdx.x == 0) {
            a.merge_tok[done_rows + at.rows] = t0;
            a.merge_ptr[done_rows + at.rows] = done_ent + at.ent;
        }
        __syncthreads();
        for (int i = blockIdx.x * kPlanThreads + tid; i < tot.dec; i += gridDim.x * kPlanThreads) {
            const int k = plan_find(row_dec, nr, i);
            const int p = i - row_dec[k], pieces = row_np[k], len = row_len[k];
            const int step = 16 * (((len + 15) / 16 + pieces - 1) / pieces);   // equal pieces
            const int ent = row_ent[k];
            const int slot = ent < 0 ? -1 : (ent + p) * a.slots_per_desc;
            WorkDesc d;
            d.tok_off = 0;
            d.shape = 1;
            d.bt_row = base + k;
            d.key_begin = p * step;
            d.key_end = min((p + 1) * step, len);
            d.part = slot;
            d.tok1 = row_t0[k];
            d.klim1 = len;
            a.desc[done_dec + i] = d;
            if (ent >= 0) {
                a.merge_ent[2 * (int64_t)(ent + p)] = slot;
                a.merge_ent[2 * (int64_t)(ent + p) + 1] = 1;   // a one-token slice, query 0
            }
        }
        // the tiles this window may write: those of the rows that fit
        const int64_t room_pf = max<int64_t>(0, used_pf - done_pf);
        const int n_tiles = (int)min<int64_t>(tot.pf, room_pf);
        for (int i = blockIdx.x * kPlanThreads + tid; i < n_tiles; i += gridDim.x * kPlanThreads) {
            const int k = plan_find(row_pf, nr, i);
            const int qk = row_q[k], c = row_len[k] - qk;
            const int n = (qk + a.tile_tokens - 1) / a.tile_tokens;
            const int first = (n - 1 - (i - row_pf[k])) * a.tile_tokens;   // most keys first
            PrefillDesc d;
            d.row = base + k;
            d.tok0 = row_t0[k] + first;
            d.ntok = min(a.tile_tokens, qk - first);
            d.key_end = c + first + d.ntok;
            d.key_begin = 0;
            d.part = -1;
            d.kfull = d.key_end - d.ntok + 1;
            d.next = 0;
            a.pdesc[done_pf + i] = d;
        }
        done_dec += tot.dec;
        done_rows += tot.rows;
        done_ent += tot.ent;
        done_pf += tot.pf;
        __syncthreads();   // the window's arrays are rewritten
    }
    if (tid == 0 && blockIdx.x == 0) {
        a.hdr[kHdrDesc] = done_dec;
        a.hdr[kHdrPdesc] = used_pf;
        a.hdr[kHdrMergeRows] = done_rows;
        a.hdr[kHdrSlots] = done_ent * a.slots_per_desc;
        a.hdr[kHdrBadRows] = bad_rows;
        a.merge_ptr[done_rows] = done_ent;
    }
}

// Block ids that one workgroup checks by itself: 32 loads per thread, which
// cost less than a launch of a workgroup per row before it (3.7 us and a gap).
constexpr int64_t kPlanCheckIds = 32 * kPlanThreads;

hipError_t launch_dev_plan(const DevPlanArgs &a, hipStream_t s) {
    if (a.num_rows <= 0) return hipSuccess;
    const int64_t width = ((int64_t)a.max_seq_len + 15) / 16;
    if (a.num_rows <= kPlanThreads && a.num_rows * width <= kPlanCheckIds) {
        hipLaunchKernelGGL((dev_plan_kernel<true>), dim3(1), dim3(kPlanThreads), 0, s, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(dev_rows_kernel, dim3((unsigned)a.num_rows), dim3(256), 0, s, a);
    // every workgroup repeats the scan, so only as many as the writing fills
    const int64_t wg = std::min<int64_t>(64, 1 + (a.cap_desc + a.cap_pdesc) / (4 * kPlanThreads));
    hipLaunchKernelGGL((dev_plan_kernel<false>), dim3((unsigned)wg), dim3(kPlanThreads), 0, s, a);
    return hipGetLastError();
}

// ----------------------------------------------------------- static scratch
//
// Device memory of echo_attn_mixed_static: the plan and partial results of
// a device-planned call live here instead of in a caller's workspace.  Each
// GPU the library runs on holds its own copy for the life of the process.
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

// Address of this device's copy of `scratch`, looked up once per device
// with that device current (in host code the array's name is not a device
// address).
hipError_t scratch_region(void **ptr) {
    static std::atomic<void *> addr[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    void *p = addr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev].store(p, std::memory_order_release);
    }
    *ptr = p;
    return hipSuccess;
}

// ------------------------------------------------------------- plan upload
//
// Copies the packed plan from pinned, coherent host memory into the
// workspace.  A kernel on the stream avoids the copy engine's hand-off with
// the kernels around it.
__global__ __launch_bounds__(256) void plan_upload_kernel(const uint32_t *__restrict__ src,
                                                          uint32_t *__restrict__ dst, int64_t words) {
    copy_words(src, dst, words, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------ launchers

hipError_t launch_append(const AppendArgs &a, int head_dim, bool fp8, hipStream_t s) {
    if (a.n_units == 0) return hipSuccess;
    const dim3 block(256);
    if (a.blocks_per_row > 0) {   // direct form: one wave per padded (row, block, head)
        const int64_t units = (int64_t)a.num_rows * a.blocks_per_row * a.num_kv_heads;
        AppendArgs d = a;
        d.n_units = units;
        const dim3 grid((unsigned)((units + 3) / 4));
        if (head_dim == 64 && !fp8) hipLaunchKernelGGL((append_rows_kernel<64, false>), grid, block, 0, s, d);
        else if (head_dim == 64) hipLaunchKernelGGL((append_rows_kernel<64, true>), grid, block, 0, s, d);
        else if (!fp8) hipLaunchKernelGGL((append_rows_kernel<128, false>), grid, block, 0, s, d);
        else hipLaunchKernelGGL((append_rows_kernel<128, true>), grid, block, 0, s, d);
        return hipGetLastError();
    }
    // (a launch holds fewer than 2^32 threads in x)
    const int64_t wg = (a.n_units + 3) / 4, gx = std::min<int64_t>(wg, 1 << 22);
    const dim3 grid((unsigned)gx, (unsigned)((wg + gx - 1) / gx));
    if (head_dim == 64 && !fp8) hipLaunchKernelGGL((append_kernel<64, false>), grid, block, 0, s, a);
    else if (head_dim == 64) hipLaunchKernelGGL((append_kernel<64, true>), grid, block, 0, s, a);
    else if (!fp8) hipLaunchKernelGGL((append_kernel<128, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((append_kernel<128, true>), grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_plan_upload(const void *src, void *dst, int64_t words, hipStream_t s) {
    if (words == 0) return hipSuccess;
    const int64_t wg = std::min<int64_t>((words / 4 + 255) / 256 + 1, 256);
    hipLaunchKernelGGL(plan_upload_kernel, dim3((unsigned)wg), dim3(256), 0, s,
                       (const uint32_t *)src, (uint32_t *)dst, words);
    return hipGetLastError();
}

hipError_t launch_block_copy(const BlockCopyArgs &a, hipStream_t s) {
    if (a.n_pairs == 0) return hipSuccess;
    const dim3 grid((unsigned)((int64_t)a.n_pairs * a.chunks)), block(256);
    hipLaunchKernelGGL(block_copy_kernel, grid, block, 0, s, a);
    return hipGetLastError();
}

int prefill_max_blocks(int head_dim) {
    return (kPfLdsLimit - (head_dim == 64 ? PfLds<64>::BYTES : PfLds<128>::BYTES)) / 4;
}

// The dynamic-LDS limit of kernel f, raised once per device (bit d: done on
// device d; concurrent first calls both set it, which is harmless).
static hipError_t raise_lds_limit(const void *f, std::atomic<uint64_t> &done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? (1ull << dev) : 0;
    if (!bit || !(done.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kPfLdsLimit);
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_release);
    }
    return hipSuccess;
}

template <int D, bool FP8, bool DENSE = false>
static hipError_t launch_prefill_t(const PrefillArgs &p, hipStream_t s) {
    static std::atomic<uint64_t> attr_devices{0};
    hipError_t e = raise_lds_limit((const void *)prefill_kernel<D, FP8, DENSE>, attr_devices);
    if (e != hipSuccess) return e;
    const int bytes = PfLds<D>::BYTES + 4 * p.max_blocks;
    const dim3 grid((unsigned)(8 * p.per_xcd)), block(kPfThreads);
    hipLaunchKernelGGL((prefill_kernel<D, FP8, DENSE>), grid, block, bytes, s, p);
    return hipGetLastError();
}

static_assert(2 * (PfLds<64>::BYTES + 4 * kTwoPerCuMaxBlocks) <= kPfLdsLimit, "two workgroups per CU");

hipError_t launch_prefill(const PrefillArgs &p, int head_dim, bool fp8, hipStream_t s) {
    if (p.n_logical <= 0) return hipSuccess;
    if (p.dense)
        return fp8 ? launch_prefill_t<64, true, true>(p, s) : launch_prefill_t<64, false, true>(p, s);
    if (head_dim == 64 && !fp8) return launch_prefill_t<64, false>(p, s);
    if (head_dim == 64) return launch_prefill_t<64, true>(p, s);
    if (!fp8) return launch_prefill_t<128, false>(p, s);
    return launch_prefill_t<128, true>(p, s);
}

// Merges of at most this many (token, head) pairs give each a wave whatever its
// entries: fewer waves than SIMDs x 2 (8,192 pairs of about four entries took
// 11.8 us that way against 9.7, 2,048 pairs of six the same either way).
constexpr int64_t kMergeWideWaves = 2048;

// Decode launch shape: runs of 16 workgroups, or shorter so that there are
// at least 64 runs, but never shorter than the run length the caller asks
// for in b.run_log2 (at most 32 workgroups); the grid is a multiple of 8 runs
// (logical workgroups past the end exit at once).  Returns the grid size and
// sets b.run_log2.
static int64_t decode_grid(AttnArgs &b) {
    const int64_t nwg = (b.n_waves + 3) / 4;
    const int min_log2 = std::min(std::max(b.run_log2, 0), 5);
    b.run_log2 = 4;
    while (b.run_log2 > 0 && ((int64_t)64 << b.run_log2) > nwg) --b.run_log2;
    b.run_log2 = std::max(b.run_log2, min_log2);
    const int64_t round = (int64_t)8 << b.run_log2;
    return (nwg + round - 1) / round * round;
}

hipError_t launch_decode(const AttnArgs &a, int head_dim, bool fp8, hipStream_t s) {
    if (a.n_waves <= 0) return hipSuccess;
    AttnArgs b = a;
    const int64_t wgs = decode_grid(b);
    b.copy_first = (int32_t)wgs;
    const int64_t copies = std::min<int64_t>((a.copy_words + 1023) / 1024, 16);
    const dim3 grid((unsigned)(wgs + copies)), block(256);
    if (head_dim == 64 && !fp8) hipLaunchKernelGGL((attn_kernel<64, false>), grid, block, 0, s, b);
    else if (head_dim == 64) hipLaunchKernelGGL((attn_kernel<64, true>), grid, block, 0, s, b);
    else if (!fp8) hipLaunchKernelGGL((attn_kernel<128, false>), grid, block, 0, s, b);
    else hipLaunchKernelGGL((attn_kernel<128, true>), grid, block, 0, s, b);
    return hipGetLastError();
}

hipError_t launch_merge(const MergeArgs &m, int head_dim, hipStream_t s) {
    if (m.n_rows <= 0) return hipSuccess;
    MergeArgs b = m;
    if (m.n_rows * m.num_q_heads <= kMergeWideWaves) b.n_wide = m.n_rows;
    b.n_waves = b.n_wide * m.num_q_heads + (m.n_rows - b.n_wide) * ((m.num_q_heads + 3) / 4);
    const dim3 grid((unsigned)((b.n_waves + 3) / 4)), block(256);
    if (head_dim == 64) hipLaunchKernelGGL((merge_kernel<64>), grid, block, 0, s, b);
    else hipLaunchKernelGGL((merge_kernel<128>), grid, block, 0, s, b);
    return hipGetLastError();
}

}  // namespace echo
