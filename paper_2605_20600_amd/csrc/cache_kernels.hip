// HIP kernels of the compressed cache, written for gfx950 (CDNA4: 64-lane
// wavefronts, 160 KB LDS per CU, 8 XCDs).
//
//   k_prefill  Step 1 cache prefilling (Sec. 4): conditional keys/values into
//              rows 0..C-1 of every head, layer state reset.
//   k_append   cache append (Sec. 3, KV Cache) + running sum of the queries of
//              the current update window (Eq. 6 is linear in the queries);
//              also fused into k_update and the attention kernels.
//   k_score    head grouping (Sec. 4, Step 2), fp64.
//   k_budgets  per-head budgets (Sec. 5.1, Implementation Details).
//   k_update   periodic update (Eqs. 2-6): sliding window (Eq. 3) or
//              Stratified Token Eviction (Eqs. 4-6), fused with the
//              compaction of the head's slots or, at the grouping step, with
//              the move into the head's own segment.
//   k_export   retained-position masks for parity checks.
//
// Everything that decides an index (grouping mass, eviction scores) is
// computed in fp64 with one fixed summation order, so the decisions do not
// depend on thread scheduling; multiplies and adds stay separate wherever a
// product can round (the attention-sum logits multiply two bf16 values, exact
// in fp64, and use fma).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "../../include/headkv.h"
#include "attn_block.h"
#include "device_common.h"
#include "layout.h"

namespace headkv {
namespace {

using namespace dev;

// ------------------------------------------------------------------ prefill
__global__ __launch_bounds__(kBlock) void k_prefill(LayerDev L, int C, int d, const uint16_t* kc,
                                                    const uint16_t* vc, int64_t seg_bytes,
                                                    int dense_cap, int dense_chunks) {
    prefill_head(L, blockIdx.x, gridDim.x, C, d, kc, vc, seg_bytes, dense_cap, dense_chunks, 0, C,
                 true, threadIdx.x, kBlock);
}

__global__ void k_append(LayerDev L, int C, int d, AppendArgs a) {
    const int h = blockIdx.x;
    append_token(L, C, d, h, head_len(L, h), a, threadIdx.x);
}

// ------------------------------------------------------------ head grouping
// The in-order sums read the weights in groups of kScoreRun, a group ahead of
// the additions: up to two groups before the first weight and past the last.
constexpr int kScoreRun = 16;

struct ScoreLds {
    // tile rows of the wavefronts that have any | weights (f64, padded)
    static size_t off_w(int len, int d, int r) {
        const int per = 64 * r, waves = (len + per - 1) / per;
        return (size_t)(waves < kBlock / 64 ? waves : kBlock / 64) * per * d * sizeof(uint16_t);
    }
    static size_t bytes(int len, int d, int r) {
        return off_w(len, d, r) + sizeof(double) * ((size_t)len + 4 * kScoreRun);
    }
};

// One block per head.  The normaliser and the backward mass are sums whose
// order decides n*, so one thread adds each of them in order: the launch is
// bound by those two chains of len dependent fp64 additions (3.2 and 4.4 us
// at 428 tokens) and by the round trips before them.  The reads of a chain go
// out kScoreRun values ahead of their additions (read one by one, each behind
// the LDS, the chains took three quarters of the launch), and the key rows
// arrive in LDS as whole rows, all of a tile's loads in flight at once, R rows
// per thread, so that a query value read from LDS serves R rows (read by the
// threads from memory, 16 bytes of 64 rows at a time, one round trip each).
// Launches one after the other, before and now: 256 heads of 428 tokens, d =
// 128, 39.9 -> 15.5 us (42.5 and 18.6 in a profiler's trace of single ones);
// 2,048 such heads 96 -> 72; 4 heads of 6,656 tokens 512 -> 166.
template <int D, int R>
__global__ __launch_bounds__(kBlock) void k_score(LayerDev L, const uint16_t* q, int32_t* n_star,
                                                  uint8_t* is_local, int len, double sqrt_d,
                                                  double tau, int local_window, int w_off) {
#pragma clang fp contract(off)
    constexpr int CH = D / 8, ROWB = 2 * D, PER = 64 * R;  // rows per wavefront and tile
    extern __shared__ __align__(16) unsigned char lds[];
    double* a = reinterpret_cast<double*>(lds + w_off) + 2 * kScoreRun;  // [len]
    __shared__ __align__(16) double qd[D];
    __shared__ double red[kBlock / 64];
    __shared__ double zsh;
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint16_t* K = reinterpret_cast<const uint16_t*>(L.kv + L.seg_off[h]);
    const unsigned char* tile = lds + wave * PER * ROWB;
    const uint32_t tile0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds +
                           wave * PER * ROWB;
    // this wavefront's rows; those past the end are the last again, or left as
    // they are (their logits are not kept)
    auto load_rows = [&](int r0) {
#pragma unroll
        for (int i = 0; i < R * CH; ++i) {
            if (r0 + i * (64 / CH) >= len) break;
            const int p = i * 64 + lane, row = p / CH, c = (p % CH) ^ swizzle<D>(row);
            load_to_lds(K + (size_t)min(r0 + row, len - 1) * D + c * 8, tile0 + i * 1024);
        }
    };
    int r0 = wave * PER;
    if (r0 < len) load_rows(r0);
    if (tid < D) qd[tid] = bf_f64(q[(size_t)h * D + tid]);
    if (tid < 3 * kScoreRun) a[tid < kScoreRun ? len + tid : tid - 3 * kScoreRun] = 0.0;
    __syncthreads();
    // logits q.k_j / sqrt(d), dims summed in order; the product of two bf16
    // values is exact in fp64, so an fma rounds like the multiply and the add
    double m = -INFINITY;
    for (; r0 < len; r0 += kBlock * R) {
        lds_loads_done();
        double acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = 0.0;
#pragma unroll 4
        for (int c = 0; c < CH; ++c) {
            Words<4> u[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int row = 64 * r + lane;
                u[r] = *reinterpret_cast<const Words<4>*>(tile + row * ROWB +
                                                          ((c ^ swizzle<D>(row)) << 4));
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double q0 = qd[8 * c + 2 * e], q1 = qd[8 * c + 2 * e + 1];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    acc[r] = fma(q0, (double)bf_lo(u[r].w[e]), acc[r]);
                    acc[r] = fma(q1, (double)bf_hi(u[r].w[e]), acc[r]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int j = r0 + 64 * r + lane;
            if (j >= len) continue;
            const double l = acc[r] / sqrt_d;
            a[j] = l;
            m = fmax(m, l);
        }
        if (r0 + kBlock * R < len) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the tile has been read
            load_rows(r0 + kBlock * R);
        }
    }
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
    if (lane == 0) red[wave] = m;
    __syncthreads();
    m = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    for (int j = tid; j < len; j += kBlock) a[j] = exp(a[j] - m);
    __syncthreads();
    if (wave == 0) {  // normaliser, summed over the cache in order (every lane the same)
        double z = 0.0, t[kScoreRun];
#pragma unroll
        for (int i = 0; i < kScoreRun; ++i) t[i] = a[i];
#pragma unroll 1
        for (int j = 0; j < len; j += kScoreRun) {
            double nx[kScoreRun];
#pragma unroll
            for (int i = 0; i < kScoreRun; ++i) nx[i] = a[j + kScoreRun + i];
            __builtin_amdgcn_sched_barrier(0);
            // (the zeros past the end do not change the sum)
#pragma unroll
            for (int i = 0; i < kScoreRun; ++i) z += t[i];
#pragma unroll
            for (int i = 0; i < kScoreRun; ++i) t[i] = nx[i];
        }
        if (tid == 0) zsh = z;
    }
    __syncthreads();
    const double z = zsh;
    for (int j = tid; j < len; j += kBlock) a[j] = a[j] / z;
    __syncthreads();
    if (wave == 0) {  // mass accumulated backward from the newest token
        const double* e = a + len - 1;
        double S = 0.0, t[kScoreRun];
        int ns = len;
#pragma unroll
        for (int i = 0; i < kScoreRun; ++i) t[i] = e[-i];
#pragma unroll 1
        for (int n0 = 0; n0 < len; n0 += kScoreRun) {
            double nx[kScoreRun];
#pragma unroll
            for (int i = 0; i < kScoreRun; ++i) nx[i] = e[-(n0 + kScoreRun + i)];
            __builtin_amdgcn_sched_barrier(0);
            const double S0 = S;
#pragma unroll
            for (int i = 0; i < kScoreRun; ++i) S += t[i];
            if (S >= tau) {  // reached in this group (the weights are not negative): where
                double x = S0;
                int n = 0;
#pragma unroll
                for (int i = 0; i < kScoreRun; ++i) {
                    x += t[i];
                    n += x >= tau ? 0 : 1;
                }
                ns = n0 + n + 1;
                break;
            }
#pragma unroll
            for (int i = 0; i < kScoreRun; ++i) t[i] = nx[i];
        }
        if (tid == 0) {
            const int loc = ns < local_window ? 1 : 0;
            n_star[h] = ns;
            is_local[h] = (uint8_t)loc;
            L.nstar[h] = ns;
            L.label[h] = loc;
        }
    }
}

// ------------------------------------------------------------------ budgets
// With cfg_pairs, batch rows 2i (conditional) and 2i+1 (unconditional) form a
// guidance pair and both take the labels of row 2i.
// host: nullptr, or pinned host memory, budgets then labels [BH] each, which the
// host reads once the kernel has ended: two device-to-host copies of a few
// hundred bytes took as long as the grouping kernel.
__global__ void k_budgets(LayerDev L, int H, int N, const uint8_t* is_local,
                          const int32_t* override_b, int32_t* budgets, int mode, int row_len,
                          int recent_len, int rho_num, int rho_den, int cfg_pairs,
                          int32_t* host) {
    __shared__ int n_local;
    const int b = blockIdx.x, h = threadIdx.x, idx = b * H + h;
    if (h == 0) n_local = 0;
    __syncthreads();
    const int loc = is_local[cfg_pairs ? (b & ~1) * H + h : idx] ? 1 : 0;
    if (loc) atomicAdd(&n_local, 1);
    __syncthreads();
    const long long rhoN = (long long)N * rho_num / rho_den;
    const int b_local = recent_len < N ? recent_len : N;
    int B;
    if (mode == HEADKV_BUDGET_OVERRIDE) {
        B = override_b[idx];
    } else if (mode == HEADKV_BUDGET_PAPER) {
        B = loc ? b_local : (int)(rhoN < 1 ? 1 : rhoN);
    } else {
        const int n_global = H - n_local;
        const long long rest = rhoN * H - (long long)n_local * b_local;
        const long long per = (n_global > 0 && rest > 0) ? rest / n_global : 0;
        long long bg = per / row_len * row_len;
        if (bg < b_local) bg = b_local;
        if (bg > N) bg = N;
        B = loc ? b_local : (int)bg;
    }
    budgets[idx] = B;
    L.budget[idx] = B;
    L.label[idx] = loc;
    if (host) {
        host[idx] = B;
        host[(int)(gridDim.x * blockDim.x) + idx] = loc;
    }
}

// The tables of the new layout from pinned host memory into the metadata, in
// one launch (five copies before, each longer than this).
__global__ __launch_bounds__(kBlock) void k_tables(LayerDev L, LayoutTables t, int BH) {
    const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (i < BH) {
        L.seg_off[i] = t.seg_off[i];
        L.cap[i] = t.cap[i];
        L.order[i] = t.order[i];
    }
    if (i <= BH) L.item_start[i] = t.item_start[i];
    if (i < t.n_items) L.items[i] = t.items[i];
}

// ------------------------------------------------------------------- update
// LDS of one update block, sized by the host from the largest source capacity
// of the launch (`cap`) and the number of visual positions (`N`).
// Steps of the query ring staged through LDS at a time when an update sums
// its window (Eq. 6 scores).
constexpr int kRingChunk = 64;

struct UpdateLds {
    static __host__ __device__ int words(int N) { return (N + 31) >> 5; }
    static __host__ __device__ size_t a16(size_t x) { return (x + 15) & ~(size_t)15; }
    // staged ring rows: the window's first chunk, rounded up to whole groups of
    // eight rows (read eight at a time)
    static __host__ __device__ int stage_steps(int P) { return ((P < kRingChunk ? P : kRingChunk) + 7) & ~7; }
    // bitmap | word prefix | order (u16) | evict (u8) | positions (i32) |
    // scores (f64, also two int lists) | with Eq. 6 scores and with
    // attention-sum scores of one query at a time: query (sum) (f64 [d]) |
    // with Eq. 6 scores: ring rows of the window staged for its sum (bf16
    // [min(P, kRingChunk)][d]); with attention-sum scores: weights of the cache
    // for each of the g queries of a group (f64 [g][C + cap], for groups with
    // weight_stride between the queries, and read kScoreRun * 2 past the end)
    static __host__ __device__ size_t off_wpre(int N) { return a16(4 * (size_t)words(N)); }
    static __host__ __device__ size_t off_order(int N) { return off_wpre(N) + a16(4 * (size_t)words(N)); }
    static __host__ __device__ size_t off_evict(int N, int cap) { return off_order(N) + a16(2 * (size_t)cap); }
    static __host__ __device__ size_t off_pos(int N, int cap) { return off_evict(N, cap) + a16((size_t)cap); }
    static __host__ __device__ size_t off_sig(int N, int cap) { return off_pos(N, cap) + a16(4 * (size_t)cap); }
    static __host__ __device__ size_t off_qs(int N, int cap) { return off_sig(N, cap) + a16(8 * (size_t)cap); }
    static __host__ __device__ size_t off_w(int N, int cap, int d) {
        return off_qs(N, cap) + a16(8 * (size_t)d);
    }
    // doubles between the weights of a group's queries: 4 more than a multiple
    // of the 32 doubles that the LDS banks hold, so that the 16 lanes that write
    // (or, in the normalisers, read) one row's weights fall on different banks
    // two at a time, the least for 16 doubles in steps of 4
    static __host__ __device__ int weight_stride(int C, int cap) {
        return (C + cap + 27) / 32 * 32 + 4;
    }
    static __host__ __device__ size_t bytes(int N, int cap, int d, int C, bool attn, int g, int P) {
        if (attn && g > 1)
            return off_qs(N, cap) + 8 * ((size_t)g * weight_stride(C, cap) + 2 * kScoreRun);
        return off_w(N, cap, d) +
               (attn ? a16(8 * ((size_t)C + cap)) : a16(2 * (size_t)d * stage_steps(P)));
    }
};

// Window queries scored together by the attention-sum variant: a group of up
// to 16 (the columns of an fp64 MFMA) when the period and the LDS allow at
// least 8, else one at a time.
constexpr int kQueryGroup = 16;
constexpr int kMinQueryGroup = 8;

// fp64 score -> unsigned key with the same order (-0 and +0 map to one key,
// since they compare equal).
__device__ __forceinline__ uint64_t score_key(double x) {
    if (x == 0.0) x = 0.0;
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Marks for eviction the mq lowest entries of part [lo, hi) by (score, rank):
// a radix select over the keys, 8 bits per pass from the top, that stops as
// soon as the chosen digit's bucket leaves entirely; if the exact threshold key
// is reached, the entries equal to it leave in rank order.
template <int NT>
__device__ void select_lowest(const double* sig, const uint16_t* order, uint8_t* evict, int lo,
                              int hi, int mq, int tid) {
    __shared__ uint32_t hist[256];
    __shared__ int pick[3];  // digit, entries below its bucket, bucket size
    if (mq <= 0) return;
    if (mq >= hi - lo) {
        for (int r = lo + tid; r < hi; r += NT) evict[order[r]] = 1;
        return;
    }
    uint64_t prefix = 0;  // chosen digits so far
    int want = mq;        // entries still to take at or above the prefix
    for (int shift = 56;; shift -= 8) {
        const uint64_t above = shift == 56 ? 0ull : ~0ull << (shift + 8);
        if (tid < 256) hist[tid] = 0u;
        __syncthreads();
        for (int r = lo + tid; r < hi; r += NT) {
            const uint64_t k = score_key(sig[r]);
            if ((k & above) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
        }
        __syncthreads();
        const int c = tid < 256 ? (int)hist[tid] : 0;
        int tot;
        const int ex = block_exclusive_scan<NT>(c, &tot);
        if (ex < want && want <= ex + c) {
            pick[0] = tid;
            pick[1] = ex;
            pick[2] = c;
        }
        __syncthreads();
        prefix |= (uint64_t)pick[0] << shift;
        want -= pick[1];
        const uint64_t upto = ~0ull << shift;
        if (want == pick[2]) {  // the whole bucket leaves with everything below it
            for (int r = lo + tid; r < hi; r += NT)
                if ((score_key(sig[r]) & upto) <= prefix) evict[order[r]] = 1;
            return;
        }
        if (shift == 0) {  // prefix is the exact threshold key
            int taken = 0;
            for (int r0 = lo; r0 < hi && taken < want; r0 += NT) {
                const int r = r0 + tid;
                const uint64_t k = r < hi ? score_key(sig[r]) : ~0ull;
                const int eq = (r < hi && k == prefix) ? 1 : 0;
                int t;
                const int e = block_exclusive_scan<NT>(eq, &t);
                if (eq && taken + e < want) evict[order[r]] = 1;
                taken += t;
            }
            for (int r = lo + tid; r < hi; r += NT)
                if (score_key(sig[r]) < prefix) evict[order[r]] = 1;
            return;
        }
        __syncthreads();  // hist and pick are rewritten next pass
    }
}

// The same two selections as select_lowest on parts [0, n_long) and
// [n_long, T), when T <= NT / Q: Q consecutive lanes (4 or 2) count the
// entries of an entry's part that come before it by (score, rank),
// and the entry leaves if fewer than its part's m do.  One pass over the part
// instead of up to eight radix passes with their barriers; the count grows
// with the part's size, so larger parts keep the radix select.  A part is
// ranked only if it keeps some and loses some entries (the only parts whose
// scores exist).
template <int NT, int Q>
__device__ void select_small(double* sig, const uint16_t* order, uint8_t* evict, int n_long,
                             int T, int m_long, int m_near, int tid) {
    static_assert(Q == 2 || Q == 4, "two or four lanes per entry");
    uint64_t* key = reinterpret_cast<uint64_t*>(sig);  // keys replace the scores in place
    auto part_of = [&](int r, int& lo, int& hi, int& mq) {
        const bool lng = r < n_long;
        lo = lng ? 0 : n_long;
        hi = lng ? n_long : T;
        mq = lng ? m_long : m_near;
    };
    {
        int lo, hi, mq;
        part_of(tid, lo, hi, mq);
        if (tid < T && mq > 0 && mq < hi - lo) key[tid] = score_key(sig[tid]);
    }
    __syncthreads();
    const int r = tid / Q, q = tid % Q;
    int lo, hi, mq;
    part_of(r, lo, hi, mq);
    if (r >= T || mq <= 0) return;
    if (mq >= hi - lo) {
        if (q == 0) evict[order[r]] = 1;
        return;
    }
    // entries before r count when not greater, those after when less
    const uint64_t kr = key[r];
    int c = 0;
#pragma unroll 4
    for (int j = lo + q; j < hi; j += Q) {
        const uint64_t kj = key[j];
        c += (j < r ? kj <= kr : kj < kr) ? 1 : 0;
    }
    // the Q lanes of an entry (an aligned pair or quad) are all here: summed
    // within the quad by DPP
    c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, false);  // lane ^ 1
    if (Q == 4) c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, false);  // lane ^ 2
    if (q == 0 && c < mq) evict[order[r]] = 1;
}

// The attention-sum variant of the eviction score (the oracle's
// ORC_SCORE_ATTN_SUM): for each window query p (steps max(0, step-P+1) ..
// step, from the query ring), its softmax over the cache it attended -- the
// prefix rows, then the retained tokens with position <= p in position order
// -- with logits q.k / sqrt(d) in fp64 and exp(l - max) summed in that order;
// sig[r] for the history ranks [r_lo, r_hi) accumulates the weights query by
// query, in step order.  The product of two bf16 values is exact in fp64, so
// an fma rounds exactly like the oracle's multiply and add.

// The number of visual tokens that query p sees: ranks with position <= p.
__device__ __forceinline__ int visible(const uint16_t* order, const int32_t* pos, int n, int p) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (pos[order[mid]] <= p) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// w[0] + w[1] + ... + w[len - 1] in order, the reads a group ahead of the
// additions (up to 2 * kScoreRun - 1 doubles past the end are read).  common:
// at most every lane's len, the same in all lanes (no lane checks its end
// before it).
__device__ __forceinline__ double sum_in_order(const double* w, int len, int common) {
#pragma clang fp contract(off)
    double z = 0.0, t[kScoreRun];
#pragma unroll
    for (int i = 0; i < kScoreRun; ++i) t[i] = w[i];
    int j = 0;
#pragma unroll 1
    for (; j + kScoreRun <= common; j += kScoreRun) {
        double nx[kScoreRun];
#pragma unroll
        for (int i = 0; i < kScoreRun; ++i) nx[i] = w[j + kScoreRun + i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kScoreRun; ++i) z += t[i];
#pragma unroll
        for (int i = 0; i < kScoreRun; ++i) t[i] = nx[i];
    }
    for (; j < len; ++j) z += w[j];
    return z;
}

// One query at a time (periods shorter than a group, caches whose weights for
// a group do not fit the LDS).  qd: LDS [D]; w: LDS [C + n].
template <int D>
__device__ void attention_sum_single(const LayerDev& L, const SegPtrs& S, int C, int h, int n,
                                     int r_lo, int r_hi, int step, const uint16_t* order,
                                     const int32_t* pos, double* qd, double* sig, double* w,
                                     double sqrt_d, int tid) {
#pragma clang fp contract(off)
    constexpr int WAVES = kBlock / 64;
    __shared__ double red[WAVES];
    __shared__ double msh, zsh;
    __shared__ int nvs;
    const int P = L.ring_len;
    const int p0 = step - P + 1 > 0 ? step - P + 1 : 0;
    const int lane = tid & 63, wave = tid >> 6;
    for (int r = r_lo + tid; r < r_hi; r += kBlock) sig[r] = 0.0;
    for (int p = p0; p <= step; ++p) {
        for (int i = tid; i < D; i += kBlock)
            qd[i] = bf_f64(L.qring[((size_t)h * P + p % P) * D + i]);
        if (tid == 0) nvs = visible(order, pos, n, p);
        __syncthreads();
        const int vis = C + nvs;
        double m = -INFINITY;
        for (int j = tid; j < vis; j += kBlock) {
            const uint16_t* row =
                j < C ? S.K + (size_t)j * D : S.K + (size_t)(C + order[j - C]) * D;
            const uint4* kr = reinterpret_cast<const uint4*>(row);
            // the query is read from LDS for every row: an offset of zero the
            // compiler cannot see through keeps it from hoisting all D values
            // out of the loop.  The values of the next T dims are read while
            // this T dims' products are added (a scheduling barrier keeps the
            // reads a stage ahead).
            int zo;
            asm volatile("s_mov_b32 %0, 0" : "=s"(zo));
            const double* qz = qd + zo;
            constexpr int T = 4;
            double acc = 0.0, qa[T], qb[T];
#pragma unroll
            for (int e = 0; e < T; ++e) qa[e] = qz[e];
            constexpr int HR = D / 16;  // half a row in flight at a time
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                uint4 v[HR];
#pragma unroll
                for (int c = 0; c < HR; ++c) v[c] = kr[half * HR + c];
#pragma unroll
                for (int c = 0; c < HR; ++c) {
                    const uint32_t wv[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
                    for (int st = 0; st < 8 / T; ++st) {
                        const int i0 = 8 * (half * HR + c) + st * T;  // first dim of the stage
                        if (i0 + T < D) {
#pragma unroll
                            for (int e = 0; e < T; ++e) qb[e] = qz[i0 + T + e];
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int e = 0; e < T; ++e) {
                            const int k = st * T + e;  // dim within the 16-byte chunk
                            acc = fma(qa[e],
                                      (double)((k & 1) ? bf_hi(wv[k / 2]) : bf_lo(wv[k / 2])), acc);
                        }
#pragma unroll
                        for (int e = 0; e < T; ++e) qa[e] = qb[e];
                    }
                }
            }
            const double l = acc / sqrt_d;
            w[j] = l;
            m = fmax(m, l);
        }
        for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
        if (lane == 0) red[wave] = m;
        __syncthreads();
        if (tid == 0) {
            double mx = red[0];
            for (int i = 1; i < WAVES; ++i) mx = fmax(mx, red[i]);
            msh = mx;
        }
        __syncthreads();
        for (int j = tid; j < vis; j += kBlock) w[j] = exp(w[j] - msh);
        __syncthreads();
        if (tid == 0) {  // normaliser, summed over the query's cache in order
            double z = 0.0;
            int j = 0;
            // the reads go out eight at a time, the additions stay in order
            for (; j + 8 <= vis; j += 8) {
                double t[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) t[u] = w[j + u];
#pragma unroll
                for (int u = 0; u < 8; ++u) z += t[u];
            }
            for (; j < vis; ++j) z += w[j];
            zsh = z;
        }
        __syncthreads();
        for (int r = r_lo + tid; r < r_hi && r < nvs; r += kBlock) sig[r] = sig[r] + w[C + r] / zsh;
        __syncthreads();  // qd, w, nvs, red, msh and zsh are rewritten for the next query
    }
}

// Element 4 t + kk of the 8 bf16 values of a 16-byte piece (kk = 0..3 by lane,
// t constant), in fp64.
__device__ __forceinline__ double piece_f64(const Words<4>& v, int t, int kk) {
    const uint32_t u = (kk & 2) ? v.w[2 * t + 1] : v.w[2 * t];
    return (double)((kk & 1) ? bf_hi(u) : bf_lo(u));
}

// G <= 16 queries at a time: the logits of 16 cache rows for all of them on
// the fp64 matrix cores (v_mfma_f64_16x16x4: A = 16 rows x 4 dims, B = 4 dims x
// 16 queries), D/4 steps that add the dims in order: a step rounds like four
// fused multiply-adds in order of its dims (checked bit for bit against fma
// chains on the GPU), so the logits are those of the scalar loop.  The G
// normalisers are summed by G lanes at once, each over its query's cache in
// order.  Bound by the fp64 rate (the vector ALU's too): on the vector ALU,
// with the query values read from LDS for every row, the LDS reads took 4 times
// the products (128 heads of up to 1,000 tokens, 65 queries of 128 dims: 395 ->
// 204 us per update launch; in the slowest blocks the logits take 81 us, the
// in-order sums 29, the exponentials 19).  w: LDS [G][wst] with wst >= C + n.
template <int D, int NT>
__device__ void attention_sum_group(const LayerDev& L, const SegPtrs& S, int C, int h, int n,
                                    int r_lo, int r_hi, int step, const uint16_t* order,
                                    const int32_t* pos, double* sig, double* w, int wst, int G,
                                    double sqrt_d, int tid) {
#pragma clang fp contract(off)
    typedef double f64x4_t __attribute__((ext_vector_type(4)));
    constexpr int WAVES = NT / 64, CH = D / 8;
    __shared__ double red[WAVES][kQueryGroup];
    __shared__ double msh[kQueryGroup], zsh[kQueryGroup];
    __shared__ int nvs[kQueryGroup];
    const int P = L.ring_len;
    const int p0 = step - P + 1 > 0 ? step - P + 1 : 0;
    const int lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, kk = lane >> 4;  // operand row or column, dim of a step
    for (int r = r_lo + tid; r < r_hi; r += NT) sig[r] = 0.0;
    // the keys of this wavefront's first 16 rows, the same for every group: each
    // group's last rows leave them behind in kv (rows past the group's are
    // computed and not used)
    auto row_ptr = [&](int j) {
        j = j < C + n ? j : C + n - 1;
        const int visual = C + order[j < C ? 0 : j - C];
        const int slot = j < C ? j : visual;
        return reinterpret_cast<const Words<4>*>(S.K + (size_t)slot * D);
    };
    Words<4> kv[CH];
    {
        const Words<4>* kr = row_ptr(wave * 16 + col);
#pragma unroll
        for (int c = 0; c < CH; ++c) kv[c] = kr[c];
    }
    for (int pa = p0; pa <= step; pa += G) {
        const int ng = step + 1 - pa < G ? step + 1 - pa : G;  // queries of this group
        if (tid < ng) nvs[tid] = visible(order, pos, n, pa + tid);
        // B: query col (past ng the last one again, unused), dims 4 s + kk
        double qb[D / 4];
        {
            const Words<4>* qr = reinterpret_cast<const Words<4>*>(
                L.qring + ((size_t)h * P + (pa + (col < ng ? col : ng - 1)) % P) * D);
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const Words<4> v = qr[c];
                qb[2 * c] = piece_f64(v, 0, kk);
                qb[2 * c + 1] = piece_f64(v, 1, kk);
            }
        }
        __syncthreads();
        const int rows = C + nvs[ng - 1];  // seen by the last query, the most
        const int vis = col < ng ? C + nvs[col] : 0;
        // logits of every visible row for all queries of the group, and maxima
        double m = -INFINITY;
        for (int j0 = wave * 16; j0 < rows; j0 += 16 * WAVES) {
            // each piece's place takes the next rows' piece as soon as it is used
            // (the barriers keep the loads there, a whole pass ahead of their use)
            const int jn = j0 + 16 * WAVES;
            const Words<4>* nx = row_ptr((jn < rows ? jn : wave * 16) + col);
            f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const double a0 = piece_f64(kv[c], 0, kk), a1 = piece_f64(kv[c], 1, kk);
                kv[c] = nx[c];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, qb[2 * c], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, qb[2 * c + 1], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // accumulator r: row j0 + kk + 4 r, query col
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = j0 + kk + 4 * r;
                if (j >= vis) continue;
                const double l = acc[r] / sqrt_d;
                w[(size_t)col * wst + j] = l;
                m = fmax(m, l);
            }
        }
        m = fmax(m, __shfl_xor(m, 16));
        m = fmax(m, __shfl_xor(m, 32));
        if (kk == 0) red[wave][col] = m;
        __syncthreads();
        if (tid < ng) {
            double mx = red[0][tid];
            for (int i = 1; i < WAVES; ++i) mx = fmax(mx, red[i][tid]);
            msh[tid] = mx;
        }
        __syncthreads();
        for (int g = 0; g < ng; ++g) {
            const int len = C + nvs[g];
            const double mg = msh[g];
            double* wg = w + (size_t)g * wst;
            for (int j = tid; j < len; j += NT) wg[j] = exp(wg[j] - mg);
        }
        __syncthreads();
        if (tid < ng) zsh[tid] = sum_in_order(w + (size_t)tid * wst, C + nvs[tid], C + nvs[0]);
        __syncthreads();
        for (int r = r_lo + tid; r < r_hi; r += NT) {
            double a = sig[r];
            for (int g = 0; g < ng; ++g)
                if (r < nvs[g]) a = a + w[(size_t)g * wst + C + r] / zsh[g];
            sig[r] = a;
        }
        __syncthreads();  // w, nvs, red, msh and zsh are rewritten for the next group
    }
}

// How global heads are scored: Eq. 6; attention sums, one query or a group of
// them at a time.  Separate instantiations.
constexpr int kScoresMeanLogit = 0, kScoresAttnSingle = 1, kScoresAttnGroup = 2;

// One block per head: optional append, then the periodic update of Eqs. 2-6
// (or, with `relayout`, the first update fused with the move into the head's
// new segment).  SCORES: the attention-sum scores (group: queries at a time)
// are separate instantiations, since their fp64 exp and matrix operands need
// more registers (the Eq. 6 kernel stays under 64 VGPRs: eight 256-thread
// blocks per CU).
// The update of head h by the block's NT threads (body of k_update and of the
// fused update + attention kernel); returns the head's length afterwards.
// FUSED: the block goes on to the attention, so it has the attention's 128
// VGPRs: where no K row was loaded ahead, a whole row is scored per round
// trip instead of half of one.
template <int D, int SCORES, int NT = kBlock, bool FUSED = false>
__device__ __forceinline__ int update_block(const LayerDev& L, int C, int N, const AppendArgs& a,
                                            const char* src_kv, int relayout,
                                            int64_t dense_seg_bytes, int dense_cap,
                                            int recent_len, int rs_num, int rs_den, int u,
                                            int step, int lds_cap, double sqrt_d, int group,
                                            int h) {
#pragma clang fp contract(off)
    constexpr bool ATTN_SUM = SCORES != kScoresMeanLogit;
    static_assert(NT >= 256 && NT % 64 == 0, "the radix select needs at least 256 threads");
    constexpr int kRow16 = D / 8;  // 16-byte chunks per row
    extern __shared__ __align__(16) unsigned char lds[];
    uint32_t* bm = reinterpret_cast<uint32_t*>(lds);
    int32_t* wpre = reinterpret_cast<int32_t*>(lds + UpdateLds::off_wpre(N));
    uint16_t* order = reinterpret_cast<uint16_t*>(lds + UpdateLds::off_order(N));
    uint8_t* evict = lds + UpdateLds::off_evict(N, lds_cap);
    double* sig = reinterpret_cast<double*>(lds + UpdateLds::off_sig(N, lds_cap));
    double* qs = reinterpret_cast<double*>(lds + UpdateLds::off_qs(N, lds_cap));
    int32_t* pos = reinterpret_cast<int32_t*>(lds + UpdateLds::off_pos(N, lds_cap));
    const int tid = threadIdx.x;
    const int n0 = head_len(L, h);
    const int B = L.budget[h];
    const int local = L.label[h];
    // the segment's metadata too, before the append's stores (after them, the
    // compiler can no longer read it through the scalar cache)
    const int cap_h = L.cap[h];
    const int64_t seg_h = L.seg_off[h];
    // the step's append, then the update that follows it; the update takes the
    // new token's position and query from the append's own values rather than
    // reading them back from memory
    const bool app = a.k != nullptr;
    AppendVals av;
    if (app) {
        av = append_load(D, h, a, tid);
        append_store(L, C, D, h, n0, a, av, tid);
    }
    const int n = n0 + (app ? 1 : 0);
    // Eq. (2): history = retained tokens older than the recent window
    const int w_eff = recent_len < B ? recent_len : B;
    const int T = n > w_eff ? n - w_eff : 0;
    const int keep = B - w_eff;
    const int M = T > keep ? T - keep : 0;
    if (!relayout && M == 0) {
        // every head's length is written at an update (the host's count of
        // appended tokens starts again from it)
        if (tid == 0) L.n[h] = n;
        return n;
    }
    // Eq. 6 window of a global head that evicts: steps w0..step of the query
    // ring (the step's own query, when this kernel appends it, from the
    // append's values)
    const int w0 = step - L.ring_len + 1 > 0 ? step - L.ring_len + 1 : 0;
    const int wlast = app ? step - 1 : step;  // last step read from the ring
    const bool window = !ATTN_SUM && !local && M > 0;

    const int src_cap = relayout ? dense_cap : cap_h;
    char* src_seg = relayout ? const_cast<char*>(src_kv) + (int64_t)h * dense_seg_bytes
                             : L.kv + seg_h;
    SegPtrs S = seg_ptrs(src_seg, C, src_cap, D);
    // With at most one slot per thread, thread s loads its slot's position
    // now, and, for a global head that scores (with registers for a whole row:
    // NT >= 512, or d = 64), its K row right after the positions, so that their round
    // trips overlap the ranking and the window sum.  The appended row is still
    // being stored: its position comes from the step, its row is read when it
    // is scored.
    constexpr bool kRowAhead = (NT >= 512 || D <= 64) && !ATTN_SUM;
    const bool one_slot = n <= NT;
    const int n_ahead = app ? n0 : n;
    const bool ahead = kRowAhead && window && one_slot;
    int p_own = 0;
    if (one_slot && tid < n) p_own = (app && tid == n0) ? a.step : S.pos[tid];
    // The window's first kRingChunk ring rows, loaded now so that their round
    // trip overlaps the ranking.  Every thread loads (past the window's rows,
    // and for a head without a window, the window's first piece again), so
    // that no branch holds a load: the wait for the position before them
    // then leaves them in flight.  16-byte pieces as a vector type: copies of
    // the struct type were kept in scratch memory.
    typedef unsigned int piece_t __attribute__((ext_vector_type(4)));
    constexpr int PER = (kRingChunk * kRow16 + NT - 1) / NT;
    piece_t wbuf[PER];
    {
        const int cw = wlast + 1 - w0 < kRingChunk ? wlast + 1 - w0 : kRingChunk;
        const int cn = window ? cw : 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int v0 = tid + k * NT;
            const int v = v0 < cn * kRow16 ? v0 : 0;
            wbuf[k] = reinterpret_cast<const piece_t*>(ring_slot(L, D, h, w0 + v / kRow16))[v % kRow16];
        }
    }
    uint4 krow[kRowAhead ? kRow16 : 1];

    // rank every occupied slot by its position: bitmap + prefix popcount
    const int nw = UpdateLds::words(N);
    for (int i = tid; i < nw; i += NT) bm[i] = 0u;
    for (int i = tid; i < n; i += NT) evict[i] = 0;
    __syncthreads();
    if (one_slot) {
        if (tid < n) {
            pos[tid] = p_own;
            atomicOr(&bm[p_own >> 5], 1u << (p_own & 31));
        }
    } else {
        // PB positions per thread in flight at a time (slot 0 stands in for the
        // slots past n, so that no branch holds a load)
        constexpr int PB = 4;
        for (int s0 = 0; s0 < n; s0 += PB * NT) {
            int pv[PB];
#pragma unroll
            for (int k = 0; k < PB; ++k) {
                const int s = s0 + tid + k * NT;
                pv[k] = S.pos[s < n ? s : 0];
            }
#pragma unroll
            for (int k = 0; k < PB; ++k) {
                const int s = s0 + tid + k * NT;
                if (s < n) {
                    const int p = (app && s == n0) ? a.step : pv[k];
                    pos[s] = p;
                    atomicOr(&bm[p >> 5], 1u << (p & 31));
                }
            }
        }
    }
    // the K rows go out once the positions are in (a wait for a position
    // would otherwise also wait for them); the empty asm completes the
    // position's load on every path, so that no later wait counts the rows
    asm volatile("" ::"v"(p_own));
    if (ahead && tid < n_ahead) {
        const uint4* kr = reinterpret_cast<const uint4*>(S.K + (size_t)(C + tid) * D);
#pragma unroll
        for (int c = 0; c < (kRowAhead ? kRow16 : 1); ++c) krow[c] = kr[c];
    }
    __syncthreads();
    {
        const int w0 = 2 * tid;
        const int c0 = w0 < nw ? __popc(bm[w0]) : 0;
        const int c1 = w0 + 1 < nw ? __popc(bm[w0 + 1]) : 0;
        int tot;
        const int ex = block_exclusive_scan<NT>(c0 + c1, &tot);
        if (w0 < nw) wpre[w0] = ex;
        if (w0 + 1 < nw) wpre[w0 + 1] = ex + c0;
    }
    __syncthreads();
    int r_own = -1;  // rank of this thread's slot (one slot per thread)
    for (int s = tid; s < n; s += NT) {
        const int p = pos[s];
        const int r = wpre[p >> 5] + __popc(bm[p >> 5] & ((1u << (p & 31)) - 1u));
        order[r] = (uint16_t)s;
        r_own = r;
    }
    __syncthreads();

    if (M > 0) {
        if (local) {
            // Eq. (3): sliding window, the M oldest leave
            for (int r = tid; r < M; r += NT) evict[order[r]] = 1;
        } else {
            // Eq. (5): long-range part = the oldest floor(T r_s) history tokens
            const int n_long = (int)((long long)T * rs_num / rs_den);
            const int n_near = T - n_long;
            int m_long = (M + (u & 1)) >> 1;
            int m_near = M - m_long;
            if (m_long > n_long) {
                m_near += m_long - n_long;
                m_long = n_long;
            }
            if (m_near > n_near) {
                m_long += m_near - n_near;
                m_near = n_near;
            }
            // a part is scored only if it keeps some and loses some tokens
            const bool sel_long = m_long > 0 && m_long < n_long;
            const bool sel_near = m_near > 0 && m_near < n_near;
            const int r_lo = sel_long ? 0 : n_long;
            const int r_hi = sel_near ? T : n_long;
            if constexpr (SCORES == kScoresAttnGroup) {
                attention_sum_group<D, NT>(L, S, C, h, n, r_lo, r_hi, step, order, pos, sig, qs,
                                           UpdateLds::weight_stride(C, lds_cap), group, sqrt_d, tid);
            } else if constexpr (SCORES == kScoresAttnSingle) {
                static_assert(NT == kBlock, "single queries run in 256-thread blocks");
                attention_sum_single<D>(
                    L, S, C, h, n, r_lo, r_hi, step, order, pos, qs, sig,
                    reinterpret_cast<double*>(lds + UpdateLds::off_w(N, lds_cap, D)), sqrt_d, tid);
            } else {
            // Eq. (6): mean raw logit of the past-P queries; the positive factor
            // 1/(P sqrt(d)) is dropped, the order is that of (sum q) . k, summed
            // over the dims in order in fp64.  Each thread reads half of its row's
            // 16-byte chunks together and then walks them in order.
            // the window's query sum, q_{w0} + ... + q_step in step order in
            // fp64: up to kRingChunk ring rows at a time (the first chunk loaded
            // above) are staged through LDS, then each of D threads adds its
            // dim's column
            {
                uint16_t* stage = reinterpret_cast<uint16_t*>(lds + UpdateLds::off_w(N, lds_cap, D));
                double qacc = 0.0;
                for (int c0 = w0; c0 <= wlast; c0 += kRingChunk) {
                    const int cn = wlast + 1 - c0 < kRingChunk ? wlast + 1 - c0 : kRingChunk;
                    if (c0 != w0) {
#pragma unroll
                        for (int k = 0; k < PER; ++k) {
                            const int v = tid + k * NT;
                            if (v < cn * kRow16)
                                wbuf[k] = reinterpret_cast<const piece_t*>(
                                    ring_slot(L, D, h, c0 + v / kRow16))[v % kRow16];
                        }
                    }
#pragma unroll
                    for (int k = 0; k < PER; ++k) {
                        const int v = tid + k * NT;
                        if (v < cn * kRow16) reinterpret_cast<piece_t*>(stage)[v] = wbuf[k];
                    }
                    __syncthreads();
                    // eight LDS reads in flight ahead of the in-order adds (the
                    // stage holds whole groups of eight rows; rows past cn are
                    // read and not added)
                    if (tid < D)
                        for (int j0 = 0; j0 < cn; j0 += 8) {
                            uint16_t x[8];
#pragma unroll
                            for (int j = 0; j < 8; ++j) x[j] = stage[(j0 + j) * D + tid];
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                if (j0 + j < cn) qacc = qacc + bf_f64(x[j]);
                        }
                    __syncthreads();
                }
                if (app && tid < D) qacc = qacc + bf_f64(av.qbits);
                if (tid < D) qs[tid] = qacc;
            }
            __syncthreads();
            if (ahead) {
                // thread s scores its own slot from the row it loaded
                if (tid < n && r_own >= r_lo && r_own < r_hi) {
                    if (tid >= n_ahead) {
                        const uint4* kr = reinterpret_cast<const uint4*>(S.K + (size_t)(C + tid) * D);
#pragma unroll
                        for (int c = 0; c < (kRowAhead ? kRow16 : 1); ++c) krow[c] = kr[c];
                    }
                    double acc = 0.0;
#pragma unroll
                    for (int c = 0; c < (kRowAhead ? kRow16 : 1); ++c) {
                        const uint32_t wv[4] = {krow[c].x, krow[c].y, krow[c].z, krow[c].w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            acc = acc + qs[8 * c + 2 * e] * (double)bf_lo(wv[e]);
                            acc = acc + qs[8 * c + 2 * e + 1] * (double)bf_hi(wv[e]);
                        }
                    }
                    sig[r_own] = acc;
                }
            } else {
                for (int r = r_lo + tid; r < r_hi; r += NT) {
                    const uint4* kr = reinterpret_cast<const uint4*>(S.K + (size_t)(C + order[r]) * D);
                    double acc = 0.0;
                    // half a row in flight at a time keeps the update kernel
                    // under 64 VGPRs (eight blocks per CU), which pays more
                    // than one round trip per row; the fused kernel takes the
                    // whole row unless the row loaded ahead holds registers
                    constexpr int NH = (FUSED && !kRowAhead) ? 1 : 2;
                    constexpr int HR = kRow16 / NH;
#pragma unroll
                    for (int half = 0; half < NH; ++half) {
                        uint4 v[HR];
#pragma unroll
                        for (int c = 0; c < HR; ++c) v[c] = kr[half * HR + c];
#pragma unroll
                        for (int c = 0; c < HR; ++c) {
                            const uint32_t wv[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
                            const int i0 = 8 * (half * HR + c);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                acc = acc + qs[i0 + 2 * e] * (double)bf_lo(wv[e]);
                                acc = acc + qs[i0 + 2 * e + 1] * (double)bf_hi(wv[e]);
                            }
                        }
                    }
                    sig[r] = acc;
                }
            }
            }
            __syncthreads();
            // per part, evict the m lowest by (score, position)
            if (T <= NT / 4) {
                select_small<NT, 4>(sig, order, evict, n_long, T, m_long, m_near, tid);
            } else if (T <= NT / 2) {
                select_small<NT, 2>(sig, order, evict, n_long, T, m_long, m_near, tid);
            } else {
                select_lowest<NT>(sig, order, evict, 0, n_long, m_long, tid);
                select_lowest<NT>(sig, order, evict, n_long, T, m_near, tid);
            }
        }
    }
    __syncthreads();
    const int n_new = n - M;
    int32_t* list_a = reinterpret_cast<int32_t*>(sig);
    int32_t* list_b = list_a + lds_cap;

    if (relayout) {
        // prefix rows, then kept slots in position order, into the new segment
        SegPtrs Dd = seg_ptrs(L.kv + L.seg_off[h], C, L.cap[h], D);
        const uint4* sk = reinterpret_cast<const uint4*>(S.K);
        const uint4* sv = reinterpret_cast<const uint4*>(S.V);
        uint4* dk = reinterpret_cast<uint4*>(Dd.K);
        uint4* dv = reinterpret_cast<uint4*>(Dd.V);
        for (int i = tid; i < C * kRow16; i += NT) {
            dk[i] = sk[i];
            dv[i] = sv[i];
        }
        int base = 0;
        for (int r0 = 0; r0 < n; r0 += NT) {
            const int r = r0 + tid;
            const int kf = (r < n && !evict[order[r]]) ? 1 : 0;
            int tot;
            const int ex = block_exclusive_scan<NT>(kf, &tot);
            if (kf) {
                list_a[base + ex] = order[r];
                Dd.pos[base + ex] = pos[order[r]];
            }
            base += tot;
        }
        __syncthreads();
        for (int i = tid; i < n_new * kRow16; i += NT) {
            const int j = i / kRow16, c = i - j * kRow16;
            const size_t src = (size_t)(C + list_a[j]) * kRow16 + c;
            const size_t dst = (size_t)(C + j) * kRow16 + c;
            dk[dst] = sk[src];
            dv[dst] = sv[src];
        }
    } else {
        // in place: evicted slots below n_new are refilled from kept slots at or
        // above n_new; the two sets are disjoint, so no copy reads a written row
        int nh = 0, nf = 0;
        for (int s0 = 0; s0 < n; s0 += NT) {
            const int s = s0 + tid;
            const int hf = (s < n_new && evict[s]) ? 1 : 0;
            const int ff = (s >= n_new && s < n && !evict[s]) ? 1 : 0;
            int th, tf;
            const int eh = block_exclusive_scan<NT>(hf, &th);
            const int ef = block_exclusive_scan<NT>(ff, &tf);
            if (hf) list_a[nh + eh] = s;
            if (ff) list_b[nf + ef] = s;
            nh += th;
            nf += tf;
        }
        __syncthreads();
        // the two lists have the same length when exactly M slots were
        // selected; the moves never read past either list
        nh = nh < nf ? nh : nf;
        uint4* k4 = reinterpret_cast<uint4*>(S.K);
        uint4* v4 = reinterpret_cast<uint4*>(S.V);
        for (int i = tid; i < nh * kRow16; i += NT) {
            const int j = i / kRow16, c = i - j * kRow16;
            const size_t dst = (size_t)(C + list_a[j]) * kRow16 + c;
            const size_t src = (size_t)(C + list_b[j]) * kRow16 + c;
            k4[dst] = k4[src];
            v4[dst] = v4[src];
        }
        for (int j = tid; j < nh; j += NT) S.pos[list_a[j]] = pos[list_b[j]];
    }
    if (tid == 0) L.n[h] = n_new;
    return n_new;
}

// NT threads per block: with Eq. 6 scores, 256 with more heads than CUs (eight
// blocks per CU), 1024 when each head has a CU to itself; attention-sum groups,
// 256 and 512 (two wavefronts per SIMD with their 256 VGPRs).
template <int D, int SCORES, int NT>
__global__ __launch_bounds__(NT) void k_update(LayerDev L, int C, int N, AppendArgs a,
                                               const char* src_kv, int relayout,
                                               int64_t dense_seg_bytes, int dense_cap,
                                               int recent_len, int rs_num, int rs_den, int u,
                                               int step, int lds_cap, double sqrt_d, int group) {
    update_block<D, SCORES, NT>(L, C, N, a, src_kv, relayout, dense_seg_bytes, dense_cap,
                                recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, group,
                                (int)blockIdx.x);
}

// A step's append, periodic update and attention in one launch, for layers
// whose attention runs one T-thread block per head: the block updates its
// head (Eq. 6 scores) with all its threads, then attends over the updated
// cache with the length it has just computed.  The head comes from the
// dispatch order when `order` is not null.  At most 128 VGPRs, as the
// attention kernels: 1024 / T blocks per CU.  The metadata tables the first
// loads need, the order and the appended count lead the argument list as
// plain pointers and an integer, preloaded into scalar registers at wave
// launch (the same fields of L are not read); the order is read by a vector
// load, whose wait stays on its own path.
template <int D, int T, int TPR>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4))) void k_update_attn(
    int32_t* len_n, int32_t* budget, int32_t* label, int64_t* seg_off, int32_t* cap,
    const int32_t* order, int dn, LayerDev L, int C, int N, AppendArgs a, int recent_len,
    int rs_num, int rs_den, int u, int step, int lds_cap, double sqrt_d,
    const uint16_t* __restrict__ q, float* __restrict__ out, int pad_len, float qscale) {
    LayerDev M = L;
    M.n = len_n;
    M.budget = budget;
    M.label = label;
    M.seg_off = seg_off;
    M.cap = cap;
    M.dn = dn;
    int h = (int)blockIdx.x;
    if (order != nullptr) {
        int lane0 = 0;
        asm("" : "+v"(lane0));
        h = __builtin_amdgcn_readfirstlane(order[(int)blockIdx.x + lane0]);
    }
    const int n = update_block<D, kScoresMeanLogit, T, true>(
        M, C, N, a, nullptr, 0, 0, 0, recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, 1, h);
    __syncthreads();  // the rows the update moved are read by other threads
    const AppendArgs none{};
    attn_block<D, false, T, false, TPR>(M, C, none, q, out, nullptr, 0, 0, pad_len, qscale, h,
                                        n);
}

// ------------------------------------------------------------------- export
__global__ __launch_bounds__(kBlock) void k_export(LayerDev L, int C, int d, int N, uint8_t* mask,
                                                   int32_t* count) {
    const int h = blockIdx.x, tid = threadIdx.x;
    const int n = head_len(L, h);
    SegPtrs s = seg_ptrs(L.kv + L.seg_off[h], C, L.cap[h], d);
    for (int p = tid; p < N; p += kBlock) mask[(size_t)h * N + p] = 0;
    __syncthreads();
    for (int j = tid; j < n; j += kBlock) mask[(size_t)h * N + s.pos[j]] = 1;
    if (tid == 0) count[h] = n;
}

inline int last_error() { return (int)hipGetLastError(); }

}  // namespace

int launch_prefill(const LayerDev& L, const Shape& s, const uint16_t* kc, const uint16_t* vc,
                   int64_t dense_seg_bytes, int dense_cap, int dense_chunks, void* stream) {
    hipLaunchKernelGGL(k_prefill, dim3(s.BH), dim3(kBlock), 0, (hipStream_t)stream, L, s.C, s.d,
                       kc, vc, dense_seg_bytes, dense_cap, dense_chunks);
    return last_error();
}

int launch_append(const LayerDev& L, const Shape& s, const AppendArgs& a, void* stream) {
    hipLaunchKernelGGL(k_append, dim3(s.BH), dim3(s.d), 0, (hipStream_t)stream, L, s.C, s.d, a);
    return last_error();
}

namespace {

template <int D, int R>
void score_launch(const LayerDev& L, const Shape& s, const uint16_t* q, int32_t* n_star,
                  uint8_t* is_local, int len, double sqrt_d, double tau, int local_window,
                  hipStream_t st) {
    // allow more than 64 KB of dynamic LDS (gfx950: 160 KB), once per kernel
    static const bool lds_ok = [] {
        const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_score<D, R>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize,
                                            160 * 1024) == hipSuccess;
        (void)hipGetLastError();
        return ok;
    }();
    (void)lds_ok;
    hipLaunchKernelGGL((k_score<D, R>), dim3(s.BH), dim3(kBlock), ScoreLds::bytes(len, D, R), st, L,
                       q, n_star, is_local, len, sqrt_d, tau, local_window,
                       (int)ScoreLds::off_w(len, D, R));
}

template <int D>
void score_dispatch(const LayerDev& L, const Shape& s, const uint16_t* q, int32_t* n_star,
                    uint8_t* is_local, int len, double sqrt_d, double tau, int local_window,
                    hipStream_t st) {
    // Two rows per thread while every head has a CU's LDS to itself and it
    // holds them with the weights; one (half the LDS) when blocks share a CU or
    // one row per thread covers the cache.
    if (len > kBlock && s.BH <= kCus && ScoreLds::bytes(len, D, 2) <= kUpdateLdsBudget)
        score_launch<D, 2>(L, s, q, n_star, is_local, len, sqrt_d, tau, local_window, st);
    else
        score_launch<D, 1>(L, s, q, n_star, is_local, len, sqrt_d, tau, local_window, st);
}

}  // namespace

int launch_score(const LayerDev& L, const Shape& s, const uint16_t* q, int32_t* n_star,
                 uint8_t* is_local, int len, double sqrt_d, double tau, int local_window,
                 void* stream) {
    if (s.d == 128)
        score_dispatch<128>(L, s, q, n_star, is_local, len, sqrt_d, tau, local_window,
                            (hipStream_t)stream);
    else
        score_dispatch<64>(L, s, q, n_star, is_local, len, sqrt_d, tau, local_window,
                           (hipStream_t)stream);
    return last_error();
}

int launch_budgets(const LayerDev& L, const Shape& s, const uint8_t* is_local,
                   const int32_t* override_b, int32_t* budgets, int mode, int row_len,
                   int recent_len, int rho_num, int rho_den, int cfg_pairs, int32_t* host,
                   void* stream) {
    hipLaunchKernelGGL(k_budgets, dim3(s.B), dim3(s.H), 0, (hipStream_t)stream, L, s.H, s.N,
                       is_local, override_b, budgets, mode, row_len, recent_len, rho_num, rho_den,
                       cfg_pairs, host);
    return last_error();
}

int launch_tables(const LayerDev& L, const Shape& s, const LayoutTables& t, void* stream) {
    const int n = t.n_items > s.BH + 1 ? t.n_items : s.BH + 1;
    hipLaunchKernelGGL(k_tables, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0,
                       (hipStream_t)stream, L, t, s.BH);
    return last_error();
}

namespace {

// Queries per group of the attention-sum scores: the window in the fewest
// groups of at most kQueryGroup that fit the LDS, of equal size, when there is
// room for kMinQueryGroup and the period has as many; else 1.  With more heads
// than CUs, half of the LDS if that suffices: one block's in-order sums run
// beside another's products.
int update_query_group(const Shape& s, int cap, int period) {
    if (period < kMinQueryGroup) return 1;
    auto fits = [&](size_t budget) {
        int g = kQueryGroup;
        while (g > 1 && UpdateLds::bytes(s.N, cap, s.d, s.C, true, g, period) > budget) --g;
        return g;
    };
    int g = s.BH > kCus ? fits(kUpdateLdsBudget / 2) : 1;
    if (g < kMinQueryGroup) g = fits(kUpdateLdsBudget);
    if (g < kMinQueryGroup) return 1;
    const int groups = (period + g - 1) / g;
    return (period + groups - 1) / groups;
}

}  // namespace

int launch_update(const LayerDev& L, const Shape& s, const AppendArgs& a, const char* src_kv,
                  int relayout, int64_t dense_seg_bytes, int dense_cap, int recent_len,
                  int rs_num, int rs_den, int u, int step, int lds_cap, double sqrt_d,
                  void* stream, void* ev_start, void* ev_stop) {
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0 = static_cast<hipEvent_t>(ev_start), e1 = static_cast<hipEvent_t>(ev_stop);
    const bool attn = L.attn_scores != 0;
    const int group = attn ? update_query_group(s, lds_cap, L.ring_len) : 1;
    const size_t lds = UpdateLds::bytes(s.N, lds_cap, s.d, s.C, attn, group, L.ring_len);
    // allow the update block more than 64 KB of dynamic LDS (gfx950: 160 KB)
    static const bool lds_ok = [] {
        const int max_lds = 160 * 1024;
#define HEADKV_UPDATE_FNS(D_)                                                  \
    reinterpret_cast<const void*>(&k_update<D_, kScoresMeanLogit, kBlock>),    \
        reinterpret_cast<const void*>(&k_update<D_, kScoresMeanLogit, 1024>),  \
        reinterpret_cast<const void*>(&k_update<D_, kScoresAttnSingle, kBlock>), \
        reinterpret_cast<const void*>(&k_update<D_, kScoresAttnGroup, kBlock>), \
        reinterpret_cast<const void*>(&k_update<D_, kScoresAttnGroup, 512>)
        const void* fns[] = {HEADKV_UPDATE_FNS(128), HEADKV_UPDATE_FNS(64)};
#undef HEADKV_UPDATE_FNS
        bool ok = true;
        for (const void* f : fns)
            ok = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds) ==
                     hipSuccess && ok;
        (void)hipGetLastError();
        return ok;
    }();
    (void)lds_ok;
    // a CU per head: the whole CU's threads on it
    const bool wide = s.BH <= kCus;
#define HEADKV_UPDATE(D_, S_, NT_)                                                                 \
    hipExtLaunchKernelGGL((k_update<D_, S_, NT_>), dim3(s.BH), dim3(NT_), lds, st, e0, e1, 0, L,  \
                          s.C, s.N, a, src_kv, relayout, dense_seg_bytes, dense_cap, recent_len,  \
                          rs_num, rs_den, u, step, lds_cap, sqrt_d, group)
#define HEADKV_UPDATE_D(D_)                                                  \
    if (!attn && wide) HEADKV_UPDATE(D_, kScoresMeanLogit, 1024);            \
    else if (!attn) HEADKV_UPDATE(D_, kScoresMeanLogit, kBlock);             \
    else if (group == 1) HEADKV_UPDATE(D_, kScoresAttnSingle, kBlock);       \
    else if (wide) HEADKV_UPDATE(D_, kScoresAttnGroup, 512);                 \
    else HEADKV_UPDATE(D_, kScoresAttnGroup, kBlock)
    if (s.d == 128) {
        HEADKV_UPDATE_D(128);
    } else {
        HEADKV_UPDATE_D(64);
    }
#undef HEADKV_UPDATE_D
#undef HEADKV_UPDATE
    return last_error();
}

namespace {

template <int D, int T, int TPR>
void update_attn_launch(const LayerDev& L, const Shape& s, const AppendArgs& a, int recent_len,
                        int rs_num, int rs_den, int u, int step, int lds_cap, double sqrt_d,
                        const uint16_t* q, float* out, int use_order, int pad_len, size_t lds,
                        hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    // allow more than 64 KB of dynamic LDS (gfx950: 160 KB), once per kernel
    static const bool lds_ok = [] {
        const bool ok = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_update_attn<D, T, TPR>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize,
                                            160 * 1024) == hipSuccess;
        (void)hipGetLastError();
        return ok;
    }();
    (void)lds_ok;
    const float qscale = (float)(1.4426950408889634 / sqrt_d);
    hipExtLaunchKernelGGL((k_update_attn<D, T, TPR>), dim3(s.BH), dim3(T), lds, st, e0, e1, 0,
                          L.n, L.budget, L.label, L.seg_off, L.cap,
                          use_order ? L.order : static_cast<int32_t*>(nullptr), L.dn, L, s.C, s.N,
                          a, recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, q, out,
                          pad_len, qscale);
}

template <int D, int T>
void update_attn_tpr(const LayerDev& L, const Shape& s, const AppendArgs& a, int recent_len,
                     int rs_num, int rs_den, int u, int step, int lds_cap, double sqrt_d,
                     const uint16_t* q, float* out, int use_order, int pad_len, int tpr,
                     size_t lds, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (tpr == kAttnTpr)
        update_attn_launch<D, T, kAttnTpr>(L, s, a, recent_len, rs_num, rs_den, u, step, lds_cap,
                                           sqrt_d, q, out, use_order, pad_len, lds, st, e0, e1);
    else if (tpr == kAttnTprShort)
        update_attn_launch<D, T, kAttnTprShort>(L, s, a, recent_len, rs_num, rs_den, u, step,
                                                lds_cap, sqrt_d, q, out, use_order, pad_len, lds,
                                                st, e0, e1);
    else if (tpr == kAttnTprWide)
        update_attn_launch<D, T, kAttnTprWide>(L, s, a, recent_len, rs_num, rs_den, u, step,
                                               lds_cap, sqrt_d, q, out, use_order, pad_len, lds,
                                               st, e0, e1);
    else
        update_attn_launch<D, T, kAttnTpr / 2>(L, s, a, recent_len, rs_num, rs_den, u, step,
                                               lds_cap, sqrt_d, q, out, use_order, pad_len, lds,
                                               st, e0, e1);
}

template <int D>
void update_attn_threads(const LayerDev& L, const Shape& s, const AppendArgs& a, int recent_len,
                         int rs_num, int rs_den, int u, int step, int lds_cap, double sqrt_d,
                         const uint16_t* q, float* out, int use_order, int pad_len, int threads,
                         int tpr, size_t lds, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
    if (threads == 1024)
        update_attn_tpr<D, 1024>(L, s, a, recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, q,
                                 out, use_order, pad_len, tpr, lds, st, e0, e1);
    else if (threads == 512)
        update_attn_tpr<D, 512>(L, s, a, recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, q,
                                out, use_order, pad_len, tpr, lds, st, e0, e1);
    else
        update_attn_tpr<D, 256>(L, s, a, recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, q,
                                out, use_order, pad_len, tpr, lds, st, e0, e1);
}

}  // namespace

int launch_update_attn(const LayerDev& L, const Shape& s, const AppendArgs& a, int recent_len,
                       int rs_num, int rs_den, int u, int step, int lds_cap, double sqrt_d,
                       const uint16_t* q, float* out, int use_order, int pad_len, int threads,
                       int tpr, void* stream, void* ev_start, void* ev_stop) {
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0 = static_cast<hipEvent_t>(ev_start), e1 = static_cast<hipEvent_t>(ev_stop);
    const size_t lds = UpdateLds::bytes(s.N, lds_cap, s.d, s.C, false, 1, L.ring_len);
    if (s.d == 128)
        update_attn_threads<128>(L, s, a, recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, q,
                                 out, use_order, pad_len, threads, tpr, lds, st, e0, e1);
    else
        update_attn_threads<64>(L, s, a, recent_len, rs_num, rs_den, u, step, lds_cap, sqrt_d, q,
                                out, use_order, pad_len, threads, tpr, lds, st, e0, e1);
    return last_error();
}

size_t update_lds_bytes(int N, int cap, int d, int C, bool attn_scores, int period) {
    return UpdateLds::bytes(N, cap, d, C, attn_scores, 1, period);
}

int launch_export(const LayerDev& L, const Shape& s, uint8_t* mask, int32_t* count,
                  void* stream) {
    hipLaunchKernelGGL(k_export, dim3(s.BH), dim3(kBlock), 0, (hipStream_t)stream, L, s.C, s.d,
                       s.N, mask, count);
    return last_error();
}

}  // namespace headkv
