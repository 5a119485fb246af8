// Causal self-attention over the conditional (prefix) tokens, the dense part
// of Step 1 (cache prefilling, Sec. 4): o_i = softmax(q_i K^T / sqrt(d), keys
// j <= i) V for the C prefix tokens of every (b, h), on the MFMA units of
// gfx950.
//
// A block of W wavefronts takes W * 32 queries of one head, 32 each.  The keys
// arrive in tiles of KT = 32 * SUBS: the K and V rows of the next tile go from
// memory straight into LDS (global_load_lds, 16 bytes per lane) while the
// current one is used, one barrier per tile.  The rows of a tile lie unpadded in
// LDS, their 16-byte pieces permuted within the row (swizzle in device_common.h)
// so that both operand reads are free of bank conflicts.  For each tile a
// wavefront computes
//   S^T = K_tile Q^T   32x32x16 bf16 MFMAs over d (A = key rows from LDS, B =
//                      the wavefront's query rows, held in registers), so
//                      that a lane holds 16 of the 32 scores of one query and
//                      32 keys, and the other 16 sit in lane l ^ 32;
//   online softmax     per query in fp32 (exp2 of scaled scores);
//   O^T += V^T P^T     32x32x16 bf16 MFMAs: the order of the 16 keys of a
//                      step is free as long as both operands agree, so the
//                      score accumulators, rounded to bf16, are the B operand
//                      as they stand (slot 8 half + e: key 4 half + e for e <
//                      4, else 8 + 4 half + e - 4), and the A operand takes
//                      the same keys from the V rows by two transposing LDS
//                      reads (ds_read_b64_tr_b16: four keys of one dim).
// The normaliser sums the bf16-rounded weights that multiply V.  The same
// launch stores the prefix keys and values into the cache (headkv_prefill):
// each block writes the rows of its own queries from the tiles in LDS.
//
// Long prefixes are bound inside the CU (C = 2048, 64 heads of 128: 30 % of the
// matrix cores' cycles, 45 % of the vector ALU's issue, no LDS bank conflicts;
// without the loads of the tiles it would take 24 % less, without the
// exponentials 6 %), short ones by their bytes.  Per launch, one after the other
// on several layers' buffers, with the tiles staged through registers, V read
// four 2-byte elements at a time, 32x32x8 steps and everything written through
// the L2, and now: C = 2048, 64 heads of 128 492 -> 103 us (670 TFLOP/s of causal
// products); C = 300, 320 heads of 64 38.8 -> 17.6 us; C = 128, 256 heads of 128
// 18.4 -> 10.9 us; C = 64, 512 heads of 128 20.3 -> 10.4 us (5.7 TB/s).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "../../include/headkv.h"
#include "device_common.h"
#include "layout.h"

namespace headkv {
namespace {

using namespace dev;

typedef short bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// What the kernel writes leaves as whole rows, past the L2 (non-temporal):
// written back from the L2 it takes longer than the reads (8 launches, C = 128,
// 256 heads of 128: 122 us through the L2, 108 with the cache rows past it, 92
// with the output too; 18.2 and 17.9 us for one launch and a conversion of its
// output to bf16, 17.9 and 14.5 for one launch and a decode step).
template <typename T>
__device__ __forceinline__ void nt_store(const T& v, T* p) {
    __builtin_nontemporal_store(v, p);
}

__device__ __forceinline__ bf16x8_t load8(const uint16_t* p) {
    const uint4 w = *reinterpret_cast<const uint4*>(p);
    return __builtin_bit_cast(bf16x8_t, w);
}

template <int D, int W, int SUBS>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2)))
void k_prefill_attn(LayerDev L, int nheads, const uint16_t* __restrict__ qc,
                    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
                    float* __restrict__ out, int C, float qscale, int64_t seg_bytes,
                    int dense_cap, int dense_chunks, int through_lds) {
    constexpr int KS = D / 16;           // 32x32x16 steps over d
    constexpr int MB = D / 32;           // 32-dim blocks of the output
    constexpr int CH = D / 8;            // 16-byte pieces of a row
    constexpr int KT = 32 * SUBS;        // keys of a tile
    constexpr int QT = 32 * W;      // queries of a block
    constexpr int ROWB = 2 * D;          // bytes of a row
    constexpr int NP = KT * CH / 64;     // 64-piece loads of a tile's K (or V)
    constexpr int TILEB = 2 * KT * ROWB;  // bytes of a buffer, a power of two
    // [buffer][K, V][KT][D]; one address bit tells the buffers apart (^= TILEB
    // below), also behind static LDS, if there were any
    extern __shared__ __align__(1 << 16) unsigned char lds[];
    static_assert((1 << 16) % (2 * TILEB) == 0, "a buffer is one address bit");
    const int tiles = (C + QT - 1) / QT;
    // the longest query tiles first; the tiles of a head are nheads blocks
    // apart, so with a multiple of 8 heads they share an XCD's L2
    const int tile = tiles - 1 - (int)blockIdx.x / nheads;
    const int bh = (int)blockIdx.x % nheads;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    prefill_head(L, bh, nheads, C, D, kc, vc, seg_bytes, dense_cap, dense_chunks, 0, 0, tile == 0,
                 tid, 64 * W);
    const int q0 = tile * QT + wave * 32;
    const int half = lane >> 5, j = lane & 31;  // j: this lane's query (and key row of a tile)
    const size_t base = (size_t)bh * C * D;
    const uint16_t* K = kc + base;
    const uint16_t* V = vc + base;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
    // a piece's place in its load is the lane's; the lane fetches the piece
    // that belongs there.  Rows past C: row C - 1 again (finite, masked).
    auto load_tile = [&](int kb, int buf, auto once) {
        constexpr bool ONCE = decltype(once)::value;
#pragma unroll
        for (int i0 = 0; i0 < NP; i0 += W) {
            const int i = i0 + wave;
            const int p = i * 64 + lane, row = p / CH, c = (p % CH) ^ swizzle<D>(row);
            const size_t src = (size_t)min(kb * KT + row, C - 1) * D + c * 8;
            const uint32_t dst = lds0 + (buf * 2 * KT) * ROWB + i * 1024;
            load_to_lds<ONCE>(K + src, dst);
            load_to_lds<ONCE>(V + src, dst + KT * ROWB);
        }
    };
    const int nk = (min(C, (tile + 1) * QT) + KT - 1) / KT;  // key tiles of this block
    if (tiles == 1 && nk == 1)  // no other block reads these rows (C = 64, 512 heads: -3 %)
        load_tile(0, 0, std::true_type{});
    else
        load_tile(0, 0, std::false_type{});
    // up to two tiles: one round trip for both
    if (nk == 2) load_tile(1, 1, std::false_type{});
    bf16x8_t qb[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        qb[s] = load8(qc + base + (size_t)min(q0 + j, C - 1) * D + 16 * s + 8 * half);

    f32x16_t acc[MB];
    float m = -INFINITY, lsum = 0.f;
    // m is a rounded product: from 2^32 on its last place is worth more than
    // exp2's range, and exp2(fmaf(score, qscale, -m)) of the largest score would
    // be 2^(half a last place), not 1.  While a lane's m is 2^20 or more (large)
    // the scores are rounded like m (the test costs 0 to 2 %: C = 2048, 64
    // heads of 128 93.2 -> 94.0 us; C = 300, 320 heads of 64 14.3 -> 14.4).
    bool large = false;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mb][r] = 0.f;
    const SegPtrs cache = seg_ptrs(L.kv + (int64_t)bh * seg_bytes, C, dense_cap, D);
    u32x4_t* cK = reinterpret_cast<u32x4_t*>(cache.K);
    u32x4_t* cV = reinterpret_cast<u32x4_t*>(cache.V);
    // this lane's part of the operand addresses: K row j, piece 2 s + half;
    // V rows 4 half + (lane & 15) / 4 (and 8 on), dims 16 ((lane >> 4) & 1) +
    // 4 (lane & 3) of a 32-dim block
    const int l16 = lane & 15, vrow = 4 * half + (l16 >> 2);
    const int vpiece = 2 * ((lane >> 4) & 1) + ((l16 & 3) >> 1);
    typedef __attribute__((address_space(3))) bf16x8_t* lds8_t;
    typedef __attribute__((address_space(3))) bf16x4_t* lds4_t;
    uint32_t ka[KS], va[MB][2];
#pragma unroll
    for (int s = 0; s < KS; ++s)
        ka[s] = lds0 + j * ROWB + (((2 * s + half) ^ swizzle<D>(j)) << 4);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = vrow + 8 * i;
            va[mb][i] = lds0 + KT * ROWB + row * ROWB + (l16 & 1) * 8 +
                        (((4 * mb + vpiece) ^ swizzle<D>(row)) << 4);
        }

    // one tile: the scores against its keys, then, 32 keys at a time, the
    // weights and their V rows
    auto use_tile = [&](int kb) {
        f32x16_t st[SUBS];
#pragma unroll
        for (int u = 0; u < SUBS; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) st[u][r] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int u = 0; u < SUBS; ++u)
                st[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    ((lds8_t)(uintptr_t)ka[s])[2 * u * ROWB], qb[s], st[u], 0, 0, 0);
        // four operand reads ahead of their use
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < KS * SUBS - 4; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
        if (kb * KT + KT - 1 > q0) {  // a tile on the diagonal: causal mask
#pragma unroll
            for (int u = 0; u < SUBS; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kb * KT + 32 * u + 8 * (r / 4) + 4 * half + (r & 3);
                    if (key > q0 + j) st[u][r] = -INFINITY;
                }
        }
#pragma unroll
        for (int u = 0; u < SUBS; ++u) {
            // 32 keys that all come after the queries: not even their zero
            // weights meet the V rows (which may hold infinities)
            if (u > 0 && kb * KT + 32 * u > q0 + 31) continue;
            float mx = st[u][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, st[u][r]);
            // the other half of the query's keys is in lane l ^ 32
            const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx),
                                                            false, false);
            mx = fmaxf(m, fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1])) * qscale);
            if (__builtin_amdgcn_ballot_w64(mx != m) != 0) {
                const float f = __builtin_amdgcn_exp2f(m - mx);  // m = -inf gives 0
                m = mx;
                large = __builtin_amdgcn_ballot_w64(!(fabsf(m) < 0x1p20f)) != 0;
                lsum *= f;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[mb][r] *= f;
            }
            float scale = qscale, less = m;
            if (__builtin_expect(large, 0)) {
#pragma clang fp contract(off)
#pragma unroll
                for (int r = 0; r < 16; ++r) st[u][r] = st[u][r] * qscale - m;
                scale = 1.f;
                less = 0.f;
            }
            // weights, rounded to bf16: the B operands of two steps
            bf16x8_t pb[2];
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                bf16x2_t p, one;
                p[0] = (__bf16)__builtin_amdgcn_exp2f(fmaf(st[u][r], scale, -less));
                p[1] = (__bf16)__builtin_amdgcn_exp2f(fmaf(st[u][r + 1], scale, -less));
                one[0] = one[1] = (__bf16)1.f;
                lsum = __builtin_amdgcn_fdot2_f32_bf16(p, one, lsum, false);
                pb[r / 8][r % 8] = p[0];
                pb[r / 8][r % 8 + 1] = p[1];
            }
#pragma unroll
            for (int g = 0; g < 2; ++g)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int off = (32 * u + 16 * g) * ROWB / 8;
                    const bf16x4_t a0 =
                        __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(uintptr_t)va[mb][0] + off);
                    const bf16x4_t a1 =
                        __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(uintptr_t)va[mb][1] + off);
                    const bf16x8_t a = __builtin_bit_cast(
                        bf16x8_t, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
                    acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[g], acc[mb], 0, 0, 0);
                }
        }
    };
    for (int kb = 0; kb < nk; ++kb) {
        const int buf = kb & 1;
        // this wavefront's loads of the tile are in, and after the barrier
        // every wavefront's, and all are done with the other buffer
        lds_loads_done();
        __syncthreads();
        if (nk > 2 && kb + 1 < nk) load_tile(kb + 1, buf ^ 1, std::false_type{});
        if ((kb + 1) * KT > tile * QT) {  // rows of this block's queries: into the cache
#pragma unroll
            for (int i0 = 0; i0 < NP; i0 += W) {
                const int p = (i0 + wave) * 64 + lane, row = p / CH;
                const int c = (p % CH) ^ swizzle<D>(row), key = kb * KT + row;
                const u32x4_t* src =
                    reinterpret_cast<const u32x4_t*>(lds + (buf * 2 * KT) * ROWB) + p;
                if (key < C) {
                    nt_store(src[0], cK + (size_t)key * CH + c);
                    nt_store(src[KT * CH], cV + (size_t)key * CH + c);
                }
            }
        }
        if (q0 < C && kb * KT <= q0 + 31) use_tile(kb);  // keys at or before the queries
        // the other buffer
#pragma unroll
        for (int s = 0; s < KS; ++s) ka[s] ^= TILEB;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            va[mb][0] ^= TILEB;
            va[mb][1] ^= TILEB;
        }
    }
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(lsum), __float_as_uint(lsum),
                                                    false, false);
    const float inv = 1.f / (__uint_as_float(x[0]) + __uint_as_float(x[1]));
    // accumulator r of block mb: dim 32 mb + 8 (r / 4) + 4 half + r % 4, i.e.
    // piece 8 mb + 2 (r / 4) + half of the row's 16-byte pieces
    auto piece = [&](int mb, int g) {
        return f32x4_t{acc[mb][4 * g] * inv, acc[mb][4 * g + 1] * inv, acc[mb][4 * g + 2] * inv,
                       acc[mb][4 * g + 3] * inv};
    };
    constexpr int OP = D / 4;  // pieces of an output row
    f32x4_t* o = reinterpret_cast<f32x4_t*>(out + base + (size_t)q0 * D);
    if (through_lds) {
        // this wavefront's 32 rows, the pieces permuted within the row
        __syncthreads();  // every wavefront is done with the tiles
        f32x4_t* ob = reinterpret_cast<f32x4_t*>(lds) + wave * 32 * OP;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                ob[j * OP + ((8 * mb + 2 * g + half) ^ (j & (OP - 1)))] = piece(mb, g);
        // rows other lanes of this wavefront wrote: no read moves above here
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < OP / 2; ++i) {
            const int row = (i * 64 + lane) / OP, c = lane & (OP - 1);
            const f32x4_t v = ob[row * OP + (c ^ (row & (OP - 1)))];
            if (q0 + row < C) nt_store(v, o + row * OP + c);
        }
    } else if (q0 + j < C) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int g = 0; g < 4; ++g) o[j * OP + 8 * mb + 2 * g + half] = piece(mb, g);
    }
}

inline int last_error() { return (int)hipGetLastError(); }

struct PrefillCall {
    const LayerDev& L;
    const Shape& s;
    const uint16_t *qc, *kc, *vc;
    float* out;
    int64_t dense_seg_bytes;
    int dense_cap, dense_chunks;
    hipStream_t st;
    hipEvent_t e0, e1;
};

template <int D, int W, int SUBS>
void prefill_attn_launch(const PrefillCall& c) {
    constexpr int QT = 32 * W, KT = 32 * SUBS;
    const float qscale = (float)(1.4426950408889634 / std::sqrt((double)D));
    const unsigned grid = (unsigned)((c.s.C + QT - 1) / QT) * (unsigned)c.s.BH;
    const size_t tile_bytes = (size_t)2 * KT * D * sizeof(uint16_t);
    // The output rows go through LDS to leave whole (and non-temporally: half
    // a row at a time that would be slower than through the L2, C = 128, 256
    // heads of 128: 192 us for 8 launches, 122 through the L2, 92 as whole
    // rows) unless the launch is so small that its latency counts: 32 heads of
    // 128, C = 200: 9.3 us, as whole rows 10.2; C = 300: 11.3 and 11.1; 256
    // heads, C = 64: 7.6 and 6.5.  At d = 64 whole rows are never slower.
    const int through_lds = D == 64 || (long long)c.s.BH * c.s.C >= 8192;
    const size_t out_bytes = through_lds ? (size_t)32 * W * D * sizeof(float) : 0;
    const size_t lds = std::max(tile_bytes * (c.s.C > KT ? 2 : 1), out_bytes);
    hipExtLaunchKernelGGL((k_prefill_attn<D, W, SUBS>), dim3(grid), dim3(64 * W), lds, c.st,
                          c.e0, c.e1, 0, c.L, c.s.BH, c.qc, c.kc, c.vc, c.out, c.s.C, qscale,
                          c.dense_seg_bytes, c.dense_cap, c.dense_chunks, through_lds);
}

// Wavefronts (of 32 queries) per block.  Four: the keys in LDS serve 128
// queries (C = 300, 256 heads of 128: 29.9 us, with two 35.3, with one 61.0; C
// = 2048, 64 heads: 103, 141 and 297).  Up to 128 tokens a head is one such
// block; two make two blocks of it, which is better as long as all of them are
// resident at once, two to a CU at d = 128, four at 64 (C = 77 / 128, d = 128,
// with four and with two: 256 heads 8.3 / 9.9 and 7.5 / 9.7 us, 320 heads 10.7
// / 12.9 and 13.0 / 15.7; d = 64, 512 heads 7.6 / 8.5 and 6.9 / 8.3, 1024 heads
// 10.9 / 19.9 and 12.7 / 19.4).  Up to 64 (32) tokens two (one) hold all
// queries.
template <int D>
void prefill_attn_dispatch(const PrefillCall& c) {
    const int C = c.s.C;
    if (C <= 32) prefill_attn_launch<D, 1, 1>(c);
    else if (C <= 64 || (C <= 128 && c.s.BH <= kCus * 128 / D)) prefill_attn_launch<D, 2, 2>(c);
    else prefill_attn_launch<D, 4, 2>(c);
}

}  // namespace

int launch_prefill_attn(const LayerDev& L, const Shape& s, const uint16_t* qc, const uint16_t* kc,
                        const uint16_t* vc, float* out, int64_t dense_seg_bytes, int dense_cap,
                        int dense_chunks, void* stream, void* ev_start, void* ev_stop) {
    const PrefillCall c{L, s, qc, kc, vc, out, dense_seg_bytes, dense_cap, dense_chunks,
                        (hipStream_t)stream, static_cast<hipEvent_t>(ev_start),
                        static_cast<hipEvent_t>(ev_stop)};
    if (s.d == 128) prefill_attn_dispatch<128>(c);
    else prefill_attn_dispatch<64>(c);
    return last_error();
}

}  // namespace headkv
