// Attention forward for few query rows (decode) on gfx950 (MI355X): the
// recurrence of attn_fwd.hip where a key/value head serves at most 16 query
// rows, counting every head of its group.
//
// HBM bounds it: every key and value is read once and feeds a few rows.  The
// tiled kernel gives each query head a workgroup of 64 or 128 rows, so a
// group's heads each read the cache (from L2) and nearly all rows are
// padding.  Here:
//  * One workgroup of eight waves takes all rows of a (batch, key/value head,
//    key split) as the 16 columns of v_mfma_f32_16x16x32_bf16: S^T = K Q^T,
//    O^T += V^T P^T, lane = row; rows of a group's heads are consecutive in
//    Q, O and LSE.
//  * The waves share nothing while they run: wave w takes tiles w, w + 8, ..
//    of the split's keys, with its own running max and sums, and they merge
//    once at the end, in LDS, in wave order.  No barrier in the loop.
//  * A wave's K and V tiles (8 KB each) go global -> LDS by DMA, each into a
//    buffer of its own: the next K tile is in flight during the softmax and P
//    V of this one, the next V tile during the scores.  (Four waves with rings
//    of five tiles, two waves with the same: 2-5 % slower, half as fast in a
//    grid of few workgroups.)
// B=8 Hq=32 Hkv=8 Sk=8191 D=128, kernel and merge: 128-130 us for the tiled
// kernel at any split count -> 50 us with the two splits it asked for (128
// workgroups), 45 us with four (6.0 TB/s).  A workgroup alone draws 58 GB/s.
//
// Internal to libtileattn (included by attn_fwd.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "lds_dma.h"

namespace tileattn_detail {

// Query rows per key/value head (heads of the group times queries) the
// decode kernel takes.
constexpr int DECODE_MAX_ROWS = 16;
// Workgroups of a decode launch: their threads are counted in 32 bits.
constexpr int64_t DECODE_MAX_WG = (1ll << 32) / 512 - 1;

struct DecodeArgs {
    const uint16_t *Q, *K, *V;
    // O fp32 or bf16 and LSE, or with splits the partial results of split 0;
    // split s adds s * o_split / s * l_split elements
    void *O;
    float *LSE;
    size_t o_split, l_split;
    int B, Hkv, Sq, Sk;
    int rows;        // Hq / Hkv * Sq
    int causal;
    int n_split;
    int split_keys;  // keys per split
    float c;         // scale * log2(e)
};

namespace decode {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

constexpr int NW = 8;                 // waves per workgroup
constexpr int NT = 64 * NW;
static_assert(DECODE_MAX_WG * NT < (1ll << 32), "threads of a launch");
constexpr int RING = 2;               // a K and a V tile per wave
constexpr int TILE_BYTES = 8192;
constexpr int DMA = TILE_BYTES / 1024;   // DMA instructions per tile
constexpr int ROWS = 16;
constexpr float LN2 = 0.69314718055994530942f;
constexpr float RESCALE_SLACK = 8.0f;       // as attn_fwd.hip
constexpr float RAISE_SHARE_LOG2 = -2.0f;

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// x over the four lanes l, l ^ 16, l ^ 32, l ^ 48 that hold one row
__device__ __forceinline__ float max_row(float x)
{
    u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float sum_row(float x)
{
    u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 16-byte chunk swizzles of the row-major tiles: K for 16-row ds_read_b128
// operand reads, V for transpose reads of eight rows (4 g .. +7) of 32 bytes
// per half wave
template <int D>
__device__ __forceinline__ int kswz(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D>
__device__ __forceinline__ int vswz(int r)
{
    return D == 128 ? 2 * (r & 3) + 8 * ((r >> 2) & 1) : 2 * ((r >> 1) & 3);
}

// wait for a tile with `later` (0 or 1) tiles of this wave issued after it
__device__ __forceinline__ void wait_tile(int later)
{
    if (later)
        tileattn_dma::wait_vmcnt<DMA>();
    else
        tileattn_dma::wait_vmcnt<0>();
}

template <int D, bool OBF16>
__global__ __launch_bounds__(NT, 1) void attn_decode_kernel(DecodeArgs a)
{
    constexpr int TK = TILE_BYTES / (2 * D);   // keys per tile (32 or 64)
    constexpr int KB = TK / 16;                // blocks of 16 keys
    constexpr int KK = D / 32;                 // k-steps of the scores
    constexpr int DB = D / 16;                 // blocks of O^T
    constexpr int CH = D / 8;                  // 16-byte chunks per row
    constexpr int RPI = 64 / CH;               // rows per DMA instruction
    __shared__ __attribute__((aligned(1024))) unsigned char lds[NW * RING * TILE_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c16 = lane & 15, g = lane >> 4;
    const int split = blockIdx.x % a.n_split;
    const int bh = blockIdx.x / a.n_split;
    unsigned char *const ring = lds + wave * (RING * TILE_BYTES);

    const uint16_t *kb = a.K + (size_t)bh * a.Sk * D, *vb = a.V + (size_t)bh * a.Sk * D;
    const size_t row0 = (size_t)bh * a.rows;     // the head's first row in Q, O and LSE
    const int k_lo = split * a.split_keys;
    const int k_hi = min(a.Sk, k_lo + a.split_keys);
    const int n_tiles = (k_hi - k_lo + TK - 1) / TK;
    const int mine = wave < n_tiles ? (n_tiles - wave + NW - 1) / NW : 0;   // this wave's tiles

    // keys visible to this lane's row, and to every row
    const int lim = a.causal ? min(c16, a.rows - 1) % a.Sq + a.Sk - a.Sq + 1 : a.Sk;
    const int lim_all = a.causal ? a.Sk - a.Sq + 1 : a.Sk;

    // Q as the B operand: row c16, dims 32 kk + 8 g .. +7 (rows past the last
    // read the last; they are never stored).  Loaded before the first DMA,
    // so that the compiler's wait for it covers no tile.
    bf16x8 q[KK];
    {
        const uint16_t *qp = a.Q + (row0 + min(c16, a.rows - 1)) * D + 8 * g;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            q[kk] = __builtin_bit_cast(bf16x8, *(const u32x4 *)(qp + 32 * kk));
        tileattn_dma::wait_vmcnt<0>();
    }

    // The wave's t-th K or V tile.  A lane fetches the chunk that belongs at
    // its slot: row RPI i + lrow, chunk lch ^ swizzle(row).  Both swizzles of
    // that row are those of lrow with bits of i flipped, so a few offsets
    // per lane (and a scalar for the rows) address a whole tile.  In a last
    // tile, rows past the last key re-read it (masked below): nothing outside
    // the slice is addressed.
    const int lrow = lane / CH, lch = lane % CH;
    constexpr int KV = D == 128 ? 4 : 2, VV = D == 128 ? 2 : 1;   // offsets that differ
    uint32_t ko[KV], vo[VV];
#pragma unroll
    for (int i = 0; i < KV; ++i)
        ko[i] = lrow * (2 * D) + (lch ^ kswz<D>(i * RPI + lrow)) * 16;
#pragma unroll
    for (int i = 0; i < VV; ++i)
        vo[i] = lrow * (2 * D) + (lch ^ vswz<D>(i * RPI + lrow)) * 16;
    auto dma = [&](int t, bool is_v) {
        const int key0 = k_lo + (t * NW + wave) * TK;
        const uint16_t *tile = (is_v ? vb : kb) + (size_t)key0 * D;
        const int last = min(TK, k_hi - key0) - 1;
        const tileattn_dma::u32x4s rs = tileattn_dma::buffer_rsrc(tile, (uint32_t)(last + 1) * (2 * D));
        const uint32_t to = tileattn_dma::lds_addr(ring) + (is_v ? TILE_BYTES : 0);
        if (last == TK - 1) {
#pragma unroll
            for (int i = 0; i < DMA; ++i)
                tileattn_dma::dma16_soff<true>(to + i * 1024, is_v ? vo[i % VV] : ko[i % KV], i * 1024, rs);
        } else {
#pragma unroll
            for (int i = 0; i < DMA; ++i) {
                const uint32_t o = is_v ? vo[i % VV] : ko[i % KV];
                tileattn_dma::dma16<true>(
                    to + i * 1024, min(i * RPI + lrow, last) * (2 * D) + o % (2 * D), rs);
            }
        }
    };

    f32x4 acc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
        acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f, m_trig = -INFINITY;

    if (mine > 0) {
        dma(0, false);
        dma(0, true);
    }
    for (int t = 0; t < mine; ++t) {
        const int key0 = k_lo + (t * NW + wave) * TK;
        // scores of the tile: lane holds keys 16 b + 4 g + r of row c16
        wait_tile(1);   // (its V tile is in flight)
        const unsigned char *kt = ring;
        f32x4 s[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const int r = 16 * b + c16;
                s[b] = mfma(*(const bf16x8 *)(kt + r * (2 * D) + (((4 * kk + g) ^ kswz<D>(r)) * 16)), q[kk],
                            s[b]);
            }
        }
        // (the tile's reads have returned before the DMA into its slot)
        __builtin_amdgcn_s_waitcnt(0xC07F);
        if (t + 1 < mine)
            dma(t + 1, false);

        const bool masked = key0 + TK > lim_all;   // uniform
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (masked)
                    s[b][r] = key0 + 16 * b + 4 * g + r < min(lim, k_hi) ? s[b][r] : -INFINITY;
                mx = fmaxf(mx, s[b][r]);
            }
        mx = max_row(mx);
        const float m_tile = mx == -INFINITY ? -INFINITY : mx * a.c;
        if (__builtin_amdgcn_ballot_w64(m_tile > m_trig)) {
            const float m_new = fmaxf(m_run, m_tile);
            const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int d = 0; d < DB; ++d)
                acc[d] *= alpha;
        }
        const float m_use = m_run == -INFINITY ? 0.f : m_run;
        float rowsum = 0.f;
        uint32_t pk[KB][2];
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int r = 0; r < 4; r += 2) {
                float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][r], a.c, -m_use));
                float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[b][r + 1], a.c, -m_use));
                if (masked) {   // (scale 0 makes a masked score NaN, not -inf)
                    p0 = s[b][r] == -INFINITY ? 0.f : p0;
                    p1 = s[b][r + 1] == -INFINITY ? 0.f : p1;
                }
                rowsum += p0 + p1;
                pk[b][r >> 1] = pack_bf16(p0, p1);
            }
        l_run += rowsum;
        m_trig = m_run + fminf(RESCALE_SLACK, fmaxf(0.f, RAISE_SHARE_LOG2 + __builtin_amdgcn_logf(l_run)));

        // O^T += V^T P^T: k-slot t of lane group g is key 32 ks + 4 g + t (t <
        // 4) or 32 ks + 16 + 4 g + t - 4, as the scores left the weights
        wait_tile(t + 1 < mine);
        const unsigned char *vt = ring + TILE_BYTES;
#pragma unroll
        for (int ks = 0; ks < TK / 32; ++ks) {
            const bf16x8 p = __builtin_bit_cast(
                bf16x8, u32x4{pk[2 * ks][0], pk[2 * ks][1], pk[2 * ks + 1][0], pk[2 * ks + 1][1]});
            const int r0 = 32 * ks + 4 * g + (c16 >> 2), r1 = r0 + 16;
#pragma unroll
            for (int d = 0; d < DB; ++d) {
                const int ch = 2 * d + ((c16 & 3) >> 1), in = 8 * (c16 & 1);
                const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_i16x4 *)(vt + r0 * (2 * D) + ((ch ^ vswz<D>(r0)) * 16) + in));
                const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (lds_i16x4 *)(vt + r1 * (2 * D) + ((ch ^ vswz<D>(r1)) * 16) + in));
                const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
                acc[d] = mfma(__builtin_bit_cast(bf16x8, u32x4{l2[0], l2[1], h2[0], h2[1]}), p, acc[d]);
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        if (t + 1 < mine)
            dma(t + 1, true);
    }

    // Merge the waves' results, each the softmax sums of its own keys, in
    // wave order.  (Every tile has been waited for; the first part of the LDS
    // is free once all waves are here.)
    float *const ml = (float *)lds;                       // [NW][2][ROWS]: m, l
    float *const po = (float *)(lds + 1024);              // [NW][ROWS][D]
    const float l = sum_row(l_run);
    __syncthreads();
    if (g == 0) {
        ml[(wave * 2 + 0) * ROWS + c16] = m_run;
        ml[(wave * 2 + 1) * ROWS + c16] = l;
    }
#pragma unroll
    for (int d = 0; d < DB; ++d)   // dims 16 d + 4 g .. +3; chunk q of row r at q ^ r
        *(f32x4 *)(po + (wave * ROWS + c16) * D + (((4 * d + g) ^ c16) * 4)) = acc[d];
    __syncthreads();
    for (int i = tid; i < ROWS * (D / 4); i += NT) {
        const int r = i / (D / 4), ch = i % (D / 4);
        if (r >= a.rows)
            break;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w)
            m = fmaxf(m, ml[(w * 2) * ROWS + r]);
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        float ls = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float mw = ml[(w * 2) * ROWS + r];
            const float e = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - m);
            ls += e * ml[(w * 2 + 1) * ROWS + r];
            o += e * *(const f32x4 *)(po + (w * ROWS + r) * D + ((ch ^ r) * 4));
        }
        const bool empty = !(ls > 0.f);
        o *= empty ? 0.f : 1.f / ls;
        const size_t e = (OBF16 ? 0 : (size_t)split * a.o_split) + (row0 + r) * D + 4 * ch;
        if (OBF16)
            *(u32x2 *)((uint16_t *)a.O + e) = u32x2{pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
        else
            *(f32x4 *)((float *)a.O + e) = o;
        if (ch == 0)
            a.LSE[(size_t)split * a.l_split + row0 + r] = empty ? -INFINITY : (m + log2f(ls)) * LN2;
    }
}

}  // namespace decode

// D = 64 or 128; rows <= DECODE_MAX_ROWS, workgroups <= DECODE_MAX_WG
inline hipError_t launch_attn_decode(const DecodeArgs &a, int D, bool o_bf16, hipStream_t stream)
{
    const dim3 grid(a.B * a.Hkv * a.n_split), block(decode::NT);
    if (D == 64) {
        if (o_bf16)
            hipLaunchKernelGGL((decode::attn_decode_kernel<64, true>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((decode::attn_decode_kernel<64, false>), grid, block, 0, stream, a);
    } else {
        if (o_bf16)
            hipLaunchKernelGGL((decode::attn_decode_kernel<128, true>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((decode::attn_decode_kernel<128, false>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace tileattn_detail
