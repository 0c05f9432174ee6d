// Block-aware budget (Alg. 1, last two steps) and per-head Top-K block
// lists (Sec. 3.2, Eq. 3).
//
// budget: per query head, the last-block masses are normalised to sum 1
//   (Alg. 1 normalises the pooled block scores), sorted descending and
//   prefix-summed; the first prefix reaching gamma gives the count k*+1 (Nk if
//   none, Nk for gamma >= 1), then raised to the minimum budget and capped at
//   Nk.
// select: per (proxy group, block row m), the m+1 causal candidates are sorted
//   by (score descending, index ascending); every head of the group lists the
//   first min(count_i, m+1) of them in that rank order and pads its row with
//   -1 (the per-row-ratio reading of Eq. 3 instead lists ceil(count_i (m+1) /
//   Nk), i.e. the same fraction of every row's causal blocks).
//   Rank order makes the lists of a group's heads prefixes of one another,
//   so the attention workgroups of those heads, which run side by side on
//   one XCD, fetch the same K/V blocks in the same order; blocks read close
//   together in time are shared through the L2.  On request the same sets
//   are listed by ascending block index instead (a rank table in LDS and a
//   stream compaction per head).
// Both are bound by their sorts.  Where the entries fit one wave's registers
// (wave_sort: budgets up to 1024 blocks, lists up to 2048) there are no
// barriers and no LDS traffic inside the sort; above, and for ascending lists,
// a workgroup sorts in LDS.  Selection calls, 32/8 heads, 4 groups, LDS sorts
// against wave sorts: 1024 blocks 95.4 -> 42.2 us (the lists alone are 134 MB
// of stores, 26 us at the copy rate), 512 blocks 41.0 -> 17.3, 256 blocks 26.4
// -> 14.5, 2048 blocks 270 -> 146 us.
// budget + select in one launch (Nk <= 128, rank order): in every select
//   workgroup, wave 0 sorts the row's candidates while waves 1-3 derive the
//   budgets of the group's heads by budget_kernel's own arithmetic (the same
//   sums and prefix sums in the same order over the same sorted shares), so
//   the counts and lists are those of the two launches for masses without
//   NaN.  On short sequences the second launch and its dependent wait are
//   most of the selection time.
// check_lists: one workgroup per (block row m, head i); validates a
//   caller-made list against what the attention step accepts.
#include "common.h"
#include "internal.h"

namespace pa {

// In-place bitonic sort of a[0..P) (P a power of two), ascending.
template <typename K>
__device__ void bitonic_sort_asc(K* a, int P, int tid, int nth) {
    for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = tid; t < P / 2; t += nth) {
                const int i = 2 * t - (t & (stride - 1));
                const int j = i + stride;
                const bool up = (i & size) == 0;
                const K x = a[i], y = a[j];
                if (up ? (x > y) : (x < y)) { a[i] = y; a[j] = x; }
            }
            __syncthreads();
        }
    }
}

static __host__ __device__ inline int next_pow2(int x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

// ---------------------------------------------------------------------------
// budget, any Nk: grid Hq, 1024 threads
// ---------------------------------------------------------------------------
constexpr int kBudgetThreads = 1024;
constexpr int kMaxBlocks = 8192;

__global__ __launch_bounds__(kBudgetThreads) void budget_kernel(Shape sh,
                                                                const float* __restrict__ mass,
                                                                float gamma, int min_blocks,
                                                                int* __restrict__ head_count) {
    __shared__ float a[kMaxBlocks];
    __shared__ float wtot[kBudgetThreads / 64];
    __shared__ int hit;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int i = blockIdx.x, nk = sh.mq;
    const int P = next_pow2(nk);
    const float* mrow = mass + (int64_t)i * nk;

    // total mass (fixed-order reduction)
    float part = 0.f;
    for (int n = tid; n < nk; n += kBudgetThreads) part += mrow[n];
    part = wave_sum(part);
    if (lane == 0) wtot[w] = part;
    if (tid == 0) hit = nk;
    __syncthreads();
    float total = 0.f;
    for (int j = 0; j < kBudgetThreads / 64; ++j) total += wtot[j];
    // normalised block shares, padded with -1 (sorted to the end)
    for (int n = tid; n < P; n += kBudgetThreads) a[n] = n < nk ? mrow[n] / total : -1.f;
    __syncthreads();
    // descending order = ascending order of the negated values
    for (int n = tid; n < P; n += kBudgetThreads) a[n] = -a[n];
    __syncthreads();
    bitonic_sort_asc<float>(a, P, tid, kBudgetThreads);
    // inclusive prefix sums: each thread owns E consecutive entries
    const int E = (P + kBudgetThreads - 1) / kBudgetThreads;
    const int e0 = tid * E;
    float own = 0.f;
    for (int e = 0; e < E; ++e) {
        const int n = e0 + e;
        if (n < nk) own += -a[n];
    }
    float incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    float excl_w = __shfl_up(incl, 1);
    if (lane == 0) excl_w = 0.f;
    __syncthreads();
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    float base = 0.f;
    for (int j = 0; j < w; ++j) base += wtot[j];
    float run = base + excl_w;
    if (gamma < 1.f) {
        for (int e = 0; e < E; ++e) {
            const int n = e0 + e;
            if (n >= nk) break;
            run += -a[n];
            if (run >= gamma) { atomicMin(&hit, n); break; }
        }
    }
    __syncthreads();
    if (tid == 0) {
        int c = (gamma < 1.f && hit < nk) ? hit + 1 : nk;
        c = max(c, min_blocks);
        c = min(c, nk);
        head_count[i] = c;
    }
}

// Lane exchange x[l ^ O] for a compile-time O: DPP for O < 16 (quad
// permutations; O = 4 as the quad reversal followed by the half-row mirror,
// since (7 - l) ^ 3 = l ^ 4 within 8 lanes; O = 8 as the row rotation by 8),
// v_permlane16_swap for 16, v_permlane32_swap for 32.
template <int O>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
    if constexpr (O == 1) {
        return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
    } else if constexpr (O == 2) {
        return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    } else if constexpr (O == 4) {
        const uint32_t y = __builtin_amdgcn_mov_dpp(x, 0x1B, 0xF, 0xF, true);  // [3,2,1,0]
        return __builtin_amdgcn_mov_dpp(y, 0x141, 0xF, 0xF, true);  // row_half_mirror
    } else if constexpr (O == 8) {
        return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true);  // row_ror:8
    } else if constexpr (O == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (__lane_id() & 16) ? r[0] : r[1];
    } else {
        static_assert(O == 32, "lane_xor: O in {1, 2, 4, 8, 16, 32}");
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (__lane_id() & 32) ? r[0] : r[1];
    }
}
template <int O>
__device__ __forceinline__ float lane_xor_f(float x) {
    return __uint_as_float(lane_xor<O>(__float_as_uint(x)));
}

// Ascending sort of 64 E distinct-or-equal values held by one wave, E per
// lane: a bitonic network whose sorted entry e = E lane + r ends in a[r] of
// the lane (the order of the input does not matter).  Strides below E stay in
// the lane's registers: a minimum and a maximum per pair.  Across lanes an
// entry takes the minimum of itself and its negated partner: the signs of the
// falling runs and of the upper lane of every pair are flipped beforehand, so
// that every exchange asks for the minimum.  One wave needs no barrier, and
// 34 of the 55 stages of 1024 entries are in registers.  K: float, or double
// for 64-bit integer keys (see row_key).
template <int O>
__device__ __forceinline__ float xor_of(float a) { return lane_xor_f<O>(a); }
template <int O>
__device__ __forceinline__ double xor_of(double a) {
    const uint64_t b = __builtin_bit_cast(uint64_t, a);
    return __builtin_bit_cast(double, ((uint64_t)lane_xor<O>((uint32_t)(b >> 32)) << 32) |
                                          lane_xor<O>((uint32_t)b));
}
__device__ __forceinline__ float flip_sign(float a, uint32_t mask) {
    return __uint_as_float(__float_as_uint(a) ^ mask);
}
__device__ __forceinline__ double flip_sign(double a, uint32_t mask) {
    return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, a) ^ ((uint64_t)mask << 32));
}
__device__ __forceinline__ float min_of(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ float max_of(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double min_of(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ double max_of(double a, double b) { return fmax(a, b); }

// sign mask of the lanes with bit L set
template <int L>
__device__ __forceinline__ uint32_t lane_sign(int lane) {
    if constexpr (L == 0 || L >= 64) return 0u;
    else return ((uint32_t)lane / L % 2) << 31;
}
template <int SIZE, int STRIDE, int E, typename K>
__device__ __forceinline__ void sort_merge(K (&a)[E], int lane, uint32_t cur) {
    // `cur`: the sign flips the entries carry
    const uint32_t dir = SIZE >= E ? lane_sign<SIZE / E>(lane) : 0u;
    if constexpr (STRIDE >= E) {
        constexpr int L = STRIDE / E;
        const uint32_t want = dir ^ lane_sign<L>(lane);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const K x = flip_sign(a[r], cur ^ want);
            a[r] = min_of(x, -xor_of<L>(x));
        }
        cur = want;
    } else {
#pragma unroll
        for (int r = 0; r < E; ++r) a[r] = flip_sign(a[r], cur ^ dir);
        cur = dir;
#pragma unroll
        for (int r = 0; r < E; ++r) {
            if ((r & STRIDE) == 0) {
                const K x = a[r], y = a[r | STRIDE];
                const bool up = SIZE >= E || (r & SIZE) == 0;
                a[r] = up ? min_of(x, y) : max_of(x, y);
                a[r | STRIDE] = up ? max_of(x, y) : min_of(x, y);
            }
        }
    }
    if constexpr (STRIDE > 1) {
        sort_merge<SIZE, STRIDE / 2>(a, lane, cur);
    } else if constexpr (SIZE < 64 * E) {
        sort_merge<SIZE * 2, SIZE>(a, lane, cur);
    } else {
#pragma unroll
        for (int r = 0; r < E; ++r) a[r] = flip_sign(a[r], cur);
    }
}
template <int E, typename K>
__device__ __forceinline__ void wave_sort(K (&a)[E], int lane) {
    sort_merge<2, 1>(a, lane, 0u);
}

// Sort key of candidate n (n < 8192) with score f: doubles in [2^52, 2^53)
// whose mantissa is (order of -score) << 13 | n, so that they order like the
// integers: ascending = score descending, index ascending.  They are distinct
// and never NaN or denormal, whatever f is.
__device__ __forceinline__ double row_key(float f, int n) {
    const uint32_t k = ~float_order_key(f);
    return __builtin_bit_cast(double, ((uint64_t)(0x43300000u | (k >> 19)) << 32) | (k << 13) |
                                          (uint32_t)n);
}
constexpr double kRowPad = 9007199254740991.0;   // 2^53 - 1: after every key
__device__ __forceinline__ int row_index(double key) {
    return (int)(__builtin_bit_cast(uint64_t, key) & 8191u);
}

// Candidates 0 .. ncand-1 (at most 64 E) of a score row in rank order, one
// wave: position p's index goes to order[p].
template <int E>
__device__ __forceinline__ void sort_row(const float* __restrict__ srow, int ncand, int lane,
                                         int* order) {
    double a[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int n = lane + 64 * r;
        a[r] = n < ncand ? row_key(srow[n], n) : kRowPad;
    }
    wave_sort<E>(a, lane);
#pragma unroll
    for (int r = 0; r < E; ++r) order[E * lane + r] = row_index(a[r]);
}

// The budgets of H heads with Nk <= 64 E in one wave, interleaved: lane l
// holds the masses x[h][r] of blocks l + 64 r (0 beyond Nk).  budget_kernel
// keeps block n in thread n (waves 0 .. E-1 with these Nk); this repeats its
// operations on the same values: each of its waves' sums of the masses,
// added in wave order (the other waves' totals are zero); the shares negated
// and sorted (padded with +1); each wave's inclusive scan, offset by the
// totals of the waves before it; and the first prefix reaching gamma.
// `tmp`: 64 E floats of this wave's own (E > 1).
template <int H, int E>
__device__ __forceinline__ void wave_budgets(const float (&x)[H][E], int nk, float gamma,
                                             int min_blocks, int lane, float* tmp, int (&c)[H]) {
    float a[H][E];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        float t[E];
#pragma unroll
        for (int r = 0; r < E; ++r) t[r] = lane + 64 * r < nk ? 0.f + x[h][r] : 0.f;
#pragma unroll
        for (int r = 0; r < E; ++r) t[r] += lane_xor_f<32>(t[r]);
#pragma unroll
        for (int r = 0; r < E; ++r) t[r] += lane_xor_f<16>(t[r]);
#pragma unroll
        for (int r = 0; r < E; ++r) t[r] += lane_xor_f<8>(t[r]);
#pragma unroll
        for (int r = 0; r < E; ++r) t[r] += lane_xor_f<4>(t[r]);
#pragma unroll
        for (int r = 0; r < E; ++r) t[r] += lane_xor_f<2>(t[r]);
#pragma unroll
        for (int r = 0; r < E; ++r) t[r] += lane_xor_f<1>(t[r]);
        float total = 0.f;
#pragma unroll
        for (int r = 0; r < E; ++r) total += t[r];
#pragma unroll
        for (int r = 0; r < E; ++r) a[h][r] = lane + 64 * r < nk ? -(x[h][r] / total) : 1.f;
    }
#pragma unroll
    for (int h = 0; h < H; ++h) wave_sort<E>(a[h], lane);
#pragma unroll
    for (int h = 0; h < H; ++h) {
        if constexpr (E > 1) {
            // entry e = E lane + r -> e = lane + 64 r
#pragma unroll
            for (int r = 0; r < E; ++r) tmp[E * lane + r] = a[h][r];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int r = 0; r < E; ++r) a[h][r] = tmp[lane + 64 * r];
            __builtin_amdgcn_wave_barrier();
        }
        float incl[E], excl[E];
#pragma unroll
        for (int r = 0; r < E; ++r) incl[r] = lane + 64 * r < nk ? 0.f + -a[h][r] : 0.f;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
            for (int r = 0; r < E; ++r) {
                const float y = __shfl_up(incl[r], o);
                if (lane >= o) incl[r] += y;
            }
        }
        float base = 0.f;
        int hit = nk;
#pragma unroll
        for (int r = 0; r < E; ++r) {
            excl[r] = __shfl_up(incl[r], 1);
            if (lane == 0) excl[r] = 0.f;
            float run = base + excl[r];
            run += -a[h][r];
            const uint64_t hits = __ballot(gamma < 1.f && lane + 64 * r < nk && run >= gamma);
            if (hit == nk && hits) hit = 64 * r + __builtin_ctzll(hits);
            base += __shfl(incl[r], 63);
        }
        int cc = (gamma < 1.f && hit < nk) ? hit + 1 : nk;
        cc = max(cc, min_blocks);
        c[h] = min(cc, nk);
    }
}

// Up to these many blocks one wave sorts a head's shares or a row's candidates
// in registers (up to 16 or 32 per lane).  Budgets stop at 1024, where
// budget_kernel's threads start to hold two blocks and its sums another order.
constexpr int kWaveBudgetBlocks = 1024;
constexpr int kWaveSortBlocks = 2048;

// budget, Nk <= 64 E <= kWaveBudgetBlocks: one wave per head (1024 blocks, 32
// heads: 20 us in budget_kernel, whose sort takes a barrier per stage; 8 us).
template <int E>
__global__ __launch_bounds__(64) void wave_budget_kernel(Shape sh, const float* __restrict__ mass,
                                                         float gamma, int min_blocks,
                                                         int* __restrict__ head_count) {
    __shared__ float tmp[64 * E];
    const int lane = threadIdx.x, i = blockIdx.x, nk = sh.mq;
    const float* mrow = mass + (int64_t)i * nk;
    float x[1][E];
    int c[1];
#pragma unroll
    for (int r = 0; r < E; ++r) x[0][r] = lane + 64 * r < nk ? mrow[lane + 64 * r] : 0.f;
    wave_budgets<1, E>(x, nk, gamma, min_blocks, lane, tmp, c);
    if (lane == 0) head_count[i] = c[0];
}

// select in rank order, Nk <= kWaveSortBlocks: one wave per (group, block
// row), four consecutive rows to a workgroup, longest rows first.  The sorted
// indices go through the wave's own LDS, so that every list is written 16
// bytes a lane (Nk a multiple of 4) in whole lines.
__global__ __launch_bounds__(256) void wave_select_kernel(Shape sh, const float* __restrict__ logA,
                                                          const int* __restrict__ head_count,
                                                          int row_ratio,
                                                          int* __restrict__ block_count,
                                                          int* __restrict__ block_index) {
    __shared__ __attribute__((aligned(16))) int order_all[4][kWaveSortBlocks];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nk = sh.mq, m = sh.mq - 1 - (4 * (int)blockIdx.x + w), g = blockIdx.y;
    if (m < 0) return;   // whole waves; no barrier follows
    int* order = order_all[w];
    const int ncand = m + 1;
    const float* srow = logA + ((int64_t)g * sh.mq + m) * nk;
    if (ncand > 1024) sort_row<32>(srow, ncand, lane, order);
    else if (ncand > 512) sort_row<16>(srow, ncand, lane, order);
    else if (ncand > 256) sort_row<8>(srow, ncand, lane, order);
    else if (ncand > 128) sort_row<4>(srow, ncand, lane, order);
    else if (ncand > 64) sort_row<2>(srow, ncand, lane, order);
    else sort_row<1>(srow, ncand, lane, order);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int i0 = g * sh.gsize, i1 = i0 + sh.gsize;
    auto kept = [&](int i) {
        const int c = min(max(head_count[i], 0), nk);   // caller-supplied: clamped
        // per-row ratio: ceil(c (m+1) / Nk), exact in integers (< 2^26)
        return row_ratio ? min((c * ncand + nk - 1) / nk, ncand) : min(c, ncand);
    };
    for (int i = i0 + lane; i < i1; i += 64) block_count[(int64_t)i * sh.mq + m] = kept(i);
    if (nk % 4 == 0) {
        typedef int i32x4 __attribute__((ext_vector_type(4)));
        for (int i = i0; i < i1; ++i) {
            const int kk = kept(i);
            int* out = block_index + ((int64_t)i * sh.mq + m) * nk;
            for (int p = 4 * lane; p < nk; p += 256) {
                i32x4 v = {-1, -1, -1, -1};
                if (p < kk) {
                    const i32x4 o = *reinterpret_cast<const i32x4*>(order + p);
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = p + u < kk ? o[u] : -1;
                }
                *reinterpret_cast<i32x4*>(out + p) = v;
            }
        }
    } else {
        for (int i = i0; i < i1; ++i) {
            const int kk = kept(i);
            int* out = block_index + ((int64_t)i * sh.mq + m) * nk;
            for (int p = lane; p < nk; p += 64) out[p] = p < kk ? order[p] : -1;
        }
    }
}

// Up to 128 blocks (two entries per lane) one launch is faster than two.
constexpr int kFusedMaxBlocks = 128;
constexpr int kFusedHeads = 3;         // heads per wave and round
constexpr int kSelectThreads = 256;

// ---------------------------------------------------------------------------
// budget and select in one launch, Nk <= 64 E <= kFusedMaxBlocks, rank order:
// grid (Mq, G), 256 threads, dynamic LDS = 4 bytes per head of the group.
// Wave 0 sorts the row's candidates while waves 1-3 derive the group's
// budgets, kFusedHeads heads per wave and round (see wave_budgets); the
// workgroups of block row 0 write the counts out.
// ---------------------------------------------------------------------------
template <int E>
__global__ __launch_bounds__(kSelectThreads) void fused_select_kernel(
    Shape sh, const float* __restrict__ logA, int* __restrict__ head_count,
    const float* __restrict__ mass, float gamma, int min_blocks, int* __restrict__ block_count,
    int* __restrict__ block_index) {
    extern __shared__ int cnt[];
    __shared__ int order[64 * E];
    __shared__ float tmp[3][64 * E];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m = blockIdx.x, g = blockIdx.y, nk = sh.mq;
    const int ncand = m + 1, i0 = g * sh.gsize, i1 = i0 + sh.gsize;
    if (w == 0) {
        sort_row<E>(logA + ((int64_t)g * sh.mq + m) * nk, ncand, lane, order);
    } else {
        for (int ib = i0 + kFusedHeads * (w - 1); ib < i1; ib += 3 * kFusedHeads) {
            float x[kFusedHeads][E];
            int c[kFusedHeads];
#pragma unroll
            for (int h = 0; h < kFusedHeads; ++h)
#pragma unroll
                for (int r = 0; r < E; ++r) {
                    const int e = lane + 64 * r;
                    x[h][r] = (ib + h < i1 && e < nk) ? mass[(int64_t)(ib + h) * nk + e] : 0.f;
                }
            wave_budgets<kFusedHeads, E>(x, nk, gamma, min_blocks, lane, tmp[w - 1], c);
            if (lane == 0) {
#pragma unroll
                for (int h = 0; h < kFusedHeads; ++h) {
                    if (ib + h < i1) {
                        cnt[ib + h - i0] = c[h];
                        if (m == 0) head_count[ib + h] = c[h];
                    }
                }
            }
        }
    }
    __syncthreads();
    // one head's list per wave at a time
    for (int i = i0 + w; i < i1; i += kSelectThreads / 64) {
        const int kk = min(cnt[i - i0], ncand);
        int* out = block_index + ((int64_t)i * sh.mq + m) * nk;
        for (int p = lane; p < nk; p += 64) out[p] = p < kk ? order[p] : -1;
        if (lane == 0) block_count[(int64_t)i * sh.mq + m] = kk;
    }
}

// ---------------------------------------------------------------------------
// select for ascending lists and for Nk > kWaveSortBlocks: grid (Mq, G), 256
// threads, dynamic LDS = P * 8 bytes (+ P * 4 for ascending lists)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSelectThreads) void select_kernel(Shape sh,
                                                                const float* __restrict__ logA,
                                                                const int* __restrict__ head_count,
                                                                int row_ratio, int ascending,
                                                                int* __restrict__ block_count,
                                                                int* __restrict__ block_index) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    __shared__ int wsum[kSelectThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m = blockIdx.x, g = blockIdx.y, nk = sh.mq;
    const int ncand = m + 1;
    const int P = next_pow2(ncand);
    uint64_t* key = reinterpret_cast<uint64_t*>(smem_raw);
    const float* srow = logA + ((int64_t)g * sh.mq + m) * nk;
    // key: (order of -score) << 32 | index  -> ascending = score desc, index asc
    for (int n = tid; n < P; n += kSelectThreads) {
        uint64_t kk = ~0ull;
        if (n < ncand) kk = ((uint64_t)(~float_order_key(srow[n])) << 32) | (uint32_t)n;
        key[n] = kk;
    }
    __syncthreads();
    bitonic_sort_asc<uint64_t>(key, P, tid, kSelectThreads);
    // ascending lists: rank[n] = position of block n in the rank order; each
    // thread owns E consecutive candidates
    int* rank = reinterpret_cast<int*>(key + P);
    const int E = (ncand + kSelectThreads - 1) / kSelectThreads;
    const int n0 = min(tid * E, ncand), n1 = min(n0 + E, ncand);
    if (ascending) {
        for (int p = tid; p < ncand; p += kSelectThreads) rank[(int)(key[p] & 0xffffffffu)] = p;
        __syncthreads();
    }
    // the sorted keys are the candidates in rank order: a head's set is the
    // first min(count, m+1) of them (sets of one group are prefixes of each
    // other); it is listed in that order, or by ascending block index
    for (int i = g * sh.gsize; i < (g + 1) * sh.gsize; ++i) {
        // counts outside [0, Nk] (caller-supplied) are clamped
        const int c = min(max(head_count[i], 0), nk);
        // per-row ratio: ceil(c (m+1) / Nk), exact in integers (< 2^26)
        const int kk = row_ratio ? min((c * ncand + nk - 1) / nk, ncand) : min(c, ncand);
        int* out = block_index + ((int64_t)i * sh.mq + m) * nk;
        if (!ascending) {
            for (int p = tid; p < nk; p += kSelectThreads)
                out[p] = p < kk ? (int)(key[p] & 0xffffffffu) : -1;
        } else {
            // stream compaction of the blocks with rank < kk, in index order:
            // a thread's own count, then an exclusive scan over the workgroup
            int own = 0;
            for (int n = n0; n < n1; ++n) own += rank[n] < kk;
            int incl = own;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            if (lane == 63) wsum[w] = incl;
            __syncthreads();
            int pos = incl - own;
            for (int j = 0; j < w; ++j) pos += wsum[j];
            for (int n = n0; n < n1; ++n)
                if (rank[n] < kk) out[pos++] = n;
            for (int p = kk + tid; p < nk; p += kSelectThreads) out[p] = -1;
            __syncthreads();   // wsum is reused by the next head
        }
        if (tid == 0) block_count[(int64_t)i * sh.mq + m] = kk;
    }
}

// Status of list (i, m): bit 0 = count outside [1, m+1]; bit 1 = one of the
// first min(max(count, 0), Nk) entries outside [0, m]; bit 2 = a block listed
// twice among them.  A bitmap of the row's m+1 causal blocks in LDS finds
// the duplicates (integer LDS atomics: the result does not depend on which
// thread sees the second copy).
constexpr int kCheckThreads = 256;

__global__ __launch_bounds__(kCheckThreads) void check_lists_kernel(
    Shape sh, const int* __restrict__ block_count, const int* __restrict__ block_index,
    int* __restrict__ status) {
    __shared__ unsigned seen[8192 / 32];
    __shared__ int flags;
    const int m = blockIdx.x, i = blockIdx.y, tid = threadIdx.x, nk = sh.mq;
    for (int wd = tid; wd < (m + 32) / 32; wd += kCheckThreads) seen[wd] = 0u;
    if (tid == 0) flags = 0;
    __syncthreads();
    const int64_t row = (int64_t)i * sh.mq + m;
    const int cnt = block_count[row];
    const int n = min(max(cnt, 0), nk);
    const int* list = block_index + row * nk;
    int f = (cnt < 1 || cnt > m + 1) ? 1 : 0;
    for (int p = tid; p < n; p += kCheckThreads) {
        const int v = list[p];
        if (v < 0 || v > m) {
            f |= 2;
        } else {
            const unsigned bit = 1u << (v & 31);
            if (atomicOr(&seen[v >> 5], bit) & bit) f |= 4;
        }
    }
    if (f) atomicOr(&flags, f);
    __syncthreads();
    if (tid == 0) status[row] = flags;
}

hipError_t launch_check_lists(const Shape& sh, const int* block_count, const int* block_index,
                              int* status, hipStream_t st) {
    hipLaunchKernelGGL(check_lists_kernel, dim3(sh.mq, sh.hq), dim3(kCheckThreads), 0, st, sh,
                       block_count, block_index, status);
    return hipGetLastError();
}

template <int E>
static void launch_wave_budget(const Shape& sh, const float* mass, float gamma, int min_blocks,
                               int* head_count, hipStream_t st) {
    hipLaunchKernelGGL(wave_budget_kernel<E>, dim3(sh.hq), dim3(64), 0, st, sh, mass, gamma,
                       min_blocks, head_count);
}

hipError_t launch_budget(const Shape& sh, const float* mass, float gamma, int min_blocks,
                         int* head_count, hipStream_t st) {
    if (sh.mq <= 64)
        launch_wave_budget<1>(sh, mass, gamma, min_blocks, head_count, st);
    else if (sh.mq <= 128)
        launch_wave_budget<2>(sh, mass, gamma, min_blocks, head_count, st);
    else if (sh.mq <= 256)
        launch_wave_budget<4>(sh, mass, gamma, min_blocks, head_count, st);
    else if (sh.mq <= 512)
        launch_wave_budget<8>(sh, mass, gamma, min_blocks, head_count, st);
    else if (sh.mq <= kWaveBudgetBlocks)
        launch_wave_budget<16>(sh, mass, gamma, min_blocks, head_count, st);
    else
        hipLaunchKernelGGL(budget_kernel, dim3(sh.hq), dim3(kBudgetThreads), 0, st, sh, mass,
                           gamma, min_blocks, head_count);
    return hipGetLastError();
}

hipError_t launch_select(const Shape& sh, const float* logA, const int* head_count,
                         int row_ratio, int ascending, int* block_count, int* block_index,
                         hipStream_t st) {
    if (!ascending && sh.mq <= kWaveSortBlocks) {
        hipLaunchKernelGGL(wave_select_kernel, dim3((sh.mq + 3) / 4, sh.g), dim3(256), 0, st, sh,
                           logA, head_count, row_ratio, block_count, block_index);
        return hipGetLastError();
    }
    const size_t P = (size_t)next_pow2(sh.mq);
    const size_t smem = P * 8 + (ascending ? P * 4 : 0);
    if (smem > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)select_kernel,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(select_kernel, dim3(sh.mq, sh.g), dim3(kSelectThreads), smem, st, sh, logA,
                       head_count, row_ratio, ascending, block_count, block_index);
    return hipGetLastError();
}

template <int E>
static hipError_t launch_fused(const Shape& sh, const float* mass, float gamma, int min_blocks,
                               int* head_count, const float* logA, int* block_count,
                               int* block_index, hipStream_t st) {
    hipLaunchKernelGGL(fused_select_kernel<E>, dim3(sh.mq, sh.g), dim3(kSelectThreads),
                       (size_t)sh.gsize * 4, st, sh, logA, head_count, mass, gamma, min_blocks,
                       block_count, block_index);
    return hipGetLastError();
}

hipError_t launch_budget_select(const Shape& sh, const float* mass, float gamma, int min_blocks,
                                int* head_count, const float* logA, int* block_count,
                                int* block_index, hipStream_t st) {
    if (sh.mq <= 64)
        return launch_fused<1>(sh, mass, gamma, min_blocks, head_count, logA, block_count,
                               block_index, st);
    if (sh.mq <= kFusedMaxBlocks)
        return launch_fused<2>(sh, mass, gamma, min_blocks, head_count, logA, block_count,
                               block_index, st);
    hipError_t e = launch_budget(sh, mass, gamma, min_blocks, head_count, st);
    if (e != hipSuccess) return e;
    return launch_select(sh, logA, head_count, 0, 0, block_count, block_index, st);
}

}  // namespace pa
