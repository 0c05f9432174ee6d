// Block scoring (Sec. 3.1, Eq. 1-2) and the last-block attention mass the
// per-head budget is read from (Alg. 1, first two steps).
//
// Proxy-head pooling (Sec. 3.1, Eq. 2 and the strided qk-pair dropping that
// follows it):
//   Q^g[t'] = fl32(sum_{i in group g, ascending} Q[s t'][i]) * fl32(1/|G|)
//   K^g[t'] = fl32(sum_{i in group g, ascending} K[s t'][kv(i)]) * fl32(1/|G|)
// rounded to nearest-even in the problem dtype.  The group's KV keys are
// summed once per query head of the group, so for GQA the pooled key is the
// mean of the KV heads of the group's query heads.  Memory-bound: each thread
// owns one 16-byte slice of one pooled row.
//
// All score tiles are computed transposed, S^T = K Q^T, on the 32x32 MFMA
// tile: lane l then owns one query (column l % 32) and 16 keys of it per
// tile, so row statistics (max, sum) are lane-local plus one exchange between
// the two wave halves.  Steps of 64 keys are copied global -> LDS without
// staging registers (double buffered, one barrier a step) and shared by the 4
// waves of a workgroup; query fragments stay in registers for the whole key
// loop.
// Bound: the VALU (per score a maximum, an FMA, an exp2 and an addition) beside
// the MFMAs, at the chip's power limit (VALU busy in 70 % and MFMA in 41 % of
// cycles at 1.8 GHz).  Against 32-key tiles staged through registers, with a
// running maximum per tile: estimate call 128K 1010 -> 942 us, 50K stride 2
// 953 -> 882 us, d 64 b 64 32K 114 -> 93 us, b 64 16K 61 -> 55 us.  Measured and
// not taken: the exponentials of the step before interleaved with the MFMAs
// (as fast), workgroups of 8 waves that halve the copies (+-2 %).
//
// Proxy scores (a2 + a3):
//   est_rowmax: one pass over the strided causal keys per strided query row,
//     giving, for every key block n <= m, the row's largest scaled logit in
//     that block, rbm[m, n][t' - m b'], and the row's (max, sum of exp2)
//     over the keys of each key chunk it covers.
//   est_reduce: combines the chunks' (max, sum) pairs into the row
//     log2-sum-exp L2[t'], then logA[m, n] = ln2 * max_{t' in m}
//     (rbm[m, n][t'] - L2[t']) = log max_{t', u'} softmax(...)  (the
//     max-pool of Eq. 1, log domain).
// A row's key range is cut into chunks of at most kEstMaxTiles 32-key tiles
// (so that no workgroup's chain of tiles sets the kernel's time), and further
// on short sequences so that the launch still fills the chip.
// One MFMA pass instead of two (no recomputation of the tiles to re-derive
// the max-pool after the row normaliser is known); rbm costs
// G * Mq(Mq+1)/2 * b' * 4 bytes of workspace.
//
// Last-block mass (a4): the last min(b, N) query tokens of every head
// against all keys, split into key chunks for parallelism, in one pass.
//   mass_block:  per (head, row, key block) the block's (max, sum of exp2).
//   mass_norm:   each row's normaliser from its blocks.
//   mass_sum:    per key block, the sum over rows of the block's share.
//
// Launches.  The two chains (pool -> est_rowmax -> est_reduce and
// mass_block -> mass_norm -> mass_sum) do not depend on each other, so each
// launch runs one stage of both, the workgroups of the two roles side by side
// in one grid (horizontal fusion: three launches instead of six, which on
// short sequences is most of the estimation time; the arithmetic of every
// output is that of the stage alone):
//   est_stage1:  pool      + mass_block
//   est_stage2:  est_rowmax + mass_norm
//   est_stage3:  est_reduce + mass_sum
// On long sequences stages 2 and 3 repeat per group of row bands, so that
// the per-(row, block) maxima they pass on need a bounded region (the mass
// stages run with the first group).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace pa {

// Keys of one step of the score kernels (one barrier each).
constexpr int kStepKeys = 64;

// Direct global -> LDS copies of the steps' key tiles: keys [64 st, 64 st +
// 64) of `base` (`ld` elements between rows), line = key - 64 st (see
// line_pos).  One instruction moves 64 consecutive 16-byte slots of the tile;
// each of the 4 waves issues INS of them, and a lane keeps one address per
// instruction, moved on by one step per copy.  Rows past the last are read
// as the last row (their scores are masked).
template <typename T, int D>
struct StepCopy {
    static constexpr int V = Vec16<T>::n;
    static constexpr int P = D / V;                      // chunks per line
    static constexpr int INS = kStepKeys * P / 64 / 4;   // instructions per wave
    static constexpr int ELEMS = kStepKeys * D;
    const T* src[INS];
    const T* base;
    int64_t ld, step_elems;
    int nrows, w, lane;

    __device__ __forceinline__ StepCopy(const T* b, int64_t ld_, int nrows_, int first_step, int w_,
                                        int lane_)
        : base(b), ld(ld_), step_elems(ld_ * kStepKeys), nrows(nrows_), w(w_), lane(lane_) {
#pragma unroll
        for (int j = 0; j < INS; ++j)
            src[j] = base + (int64_t)(first_step * kStepKeys + line(j)) * ld + chunk(j) * V;
    }
    __device__ __forceinline__ int line(int j) const { return ((w * INS + j) * 64 + lane) / P; }
    __device__ __forceinline__ int chunk(int j) const { return lane % P ^ chunk_xor<P>(line(j)); }
    // Copies step st; called for consecutive steps from first_step on.
    __device__ __forceinline__ void issue(int st, T* lds) {
        const bool whole = (st + 1) * kStepKeys <= nrows;
#pragma unroll
        for (int j = 0; j < INS; ++j) {
            const T* p = src[j];
            if (!whole) {
                const int row = min(st * kStepKeys + line(j), nrows - 1);
                p = base + (int64_t)row * ld + chunk(j) * V;
            }
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)p,
                (__attribute__((address_space(3))) void*)(lds + (w * INS + j) * 64 * V), 16, 0, 0);
            src[j] += step_elems;
        }
    }
};

// Scores of one step, transposed (64 keys x 32 queries of one wave): lane
// (lc, h) receives the keys 32 kt + c_row(r, h) of query lc.  `half`: no query
// of the wave sees a key of the second tile.  fp32 then leaves it out (its
// scores are -inf): up to 128 tokens a launch lasts as long as one step, and
// most of it is the tiles' splits and MFMAs.  Estimate call, 8/2 heads, d 128
// b 64, both tiles against this: 16 tokens 18.0 -> 15.0 us, 33 18.7 -> 17.1, 64
// 19.3 -> 17.8, 128 19.7 -> 18.0 (32-key steps 14.2, 17.2, 18.0, 18.4); longer
// ones -2 to +0.5 %.  bf16 gained 0.2 us there and at d 64 b 64 lost 4-7 % at 8K
// (stride 1, 32 heads 61.7 -> 66.0 us).
template <typename T, int D>
__device__ __forceinline__ void step_scores(f32x16 (&acc)[2], const T* tile,
                                            const LaneLines<T, D>& lines,
                                            const typename OperandOf<T>::type* qf, bool half) {
    acc[0] = zero16();
    acc[1] = zero16();
    if (sizeof(T) == 4 && half) {
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            mma(acc[0], key_operand(lines.frag(tile, 16 * ks)), qf[ks]);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[1][r] = kNegInf;
        return;
    }
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        mma(acc[0], key_operand(lines.frag(tile, 16 * ks)), qf[ks]);
        mma(acc[1], key_operand(lines.frag(tile + 32 * D, 16 * ks)), qf[ks]);
    }
}

// Keys past offset `lim` of the step (the query's last visible key) become -inf.
__device__ __forceinline__ void step_mask(f32x16 (&acc)[2], int lim, int h) {
    const int lim_h = lim - 4 * h;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            acc[kt][r] = 32 * kt + 8 * (r >> 2) + (r & 3) <= lim_h ? acc[kt][r] : kNegInf;
}

__device__ __forceinline__ float max8(const f32x16& a, int r0) {
    return fmaxf(fmaxf(fmaxf(a[r0], a[r0 + 1]), fmaxf(a[r0 + 2], a[r0 + 3])),
                 fmaxf(fmaxf(a[r0 + 4], a[r0 + 5]), fmaxf(a[r0 + 6], a[r0 + 7])));
}

// Sum of exp2(scale2 s + neg) over a step's scores: eight chains of four, then
// pairwise (as many additions as one chain, with shorter rounding paths).
__device__ __forceinline__ float step_sum(const f32x16 (&acc)[2], float scale2, float neg) {
    float c[8];
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const float x = fast_exp2(fmaf(acc[e / 16][e % 16], scale2, neg));
        c[e % 8] = e < 8 ? x : c[e % 8] + x;
    }
    return ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
}

// Slack (log2 units) by which a step's maximum may exceed the reference of a
// running sum of exp2 before the sum is rescaled: the usual step needs no
// rescaling, and the largest terms' exponents stay below 1, where their
// rounding is small (a slack of 8 raised the scores' error against 64 bits by
// 8 % and was no faster; none at all costs 0.5-1.5 %).
constexpr float kSumSlack = 1.f;

// max over both wave halves of a in lanes 0..31 and of b in lanes 32..63
__device__ __forceinline__ float halves_max2(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// ---------------------------------------------------------------------------
// a1: pooling.  One 256-thread workgroup per 256 (pooled row, 16-byte slice)
// pairs of one group; `blk` is the workgroup's index among the group's, so
// that heads are the same for the whole workgroup, their addresses scalar,
// and a KV head's slice is loaded once for the batch's query heads.  (One
// index over all groups, divided per lane, and a K load per query head: estimate
// call 128K 969 -> 962 us, 32K d 64 135 -> 132 us.  Pooling workgroups dealt
// between those of mass_block: up to 9 % slower at 50K, as fast at best.)
// ---------------------------------------------------------------------------
template <typename T, int D>
__device__ __forceinline__ void pool_body(const Shape& sh, const T* __restrict__ q,
                                          const T* __restrict__ k, T* __restrict__ qg,
                                          T* __restrict__ kg, int g, int blk) {
    constexpr int V = Vec16<T>::n;
    constexpr int SLICES = D / V;
    const int slice = threadIdx.x % SLICES;
    const int tp = blk * (256 / SLICES) + threadIdx.x / SLICES;
    if (tp >= sh.np) return;
    const int64_t t = (int64_t)tp * sh.s;
    float aq[V], ak[V];
#pragma unroll
    for (int e = 0; e < V; ++e) { aq[e] = 0.f; ak[e] = 0.f; }
    // the heads' slices are loaded kPoolBatch at a time (all in flight
    // together; a batch past the group's last head re-reads that head and
    // discards it), then added in ascending head order
    constexpr int kPoolBatch = 4;
    const int i0 = g * sh.gsize, i1 = i0 + sh.gsize;
    const T* qrow = q + t * sh.q_tok + slice * V;
    const T* krow = k + t * sh.kv_tok + slice * V;
    for (int ib = i0; ib < i1; ib += kPoolBatch) {
        uint4 qv[kPoolBatch], kv[kPoolBatch];
        // a batch's heads of one KV head share its slice: one load
        const int last = min(ib + kPoolBatch, i1) - 1;
        const bool one_kv = ib / sh.rep == last / sh.rep;
#pragma unroll
        for (int u = 0; u < kPoolBatch; ++u)
            qv[u] = *reinterpret_cast<const uint4*>(qrow + (int64_t)min(ib + u, last) * sh.q_head);
        if (one_kv) {
            kv[0] = *reinterpret_cast<const uint4*>(krow + (int64_t)(ib / sh.rep) * sh.kv_head);
#pragma unroll
            for (int u = 1; u < kPoolBatch; ++u) kv[u] = kv[0];
        } else {
#pragma unroll
            for (int u = 0; u < kPoolBatch; ++u)
                kv[u] = *reinterpret_cast<const uint4*>(
                    krow + (int64_t)(min(ib + u, last) / sh.rep) * sh.kv_head);
        }
#pragma unroll
        for (int u = 0; u < kPoolBatch; ++u) {
            if (ib + u < i1) {
                const T* qe = reinterpret_cast<const T*>(&qv[u]);
                const T* ke = reinterpret_cast<const T*>(&kv[u]);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    aq[e] = aq[e] + to_f32<T>(qe[e]);
                    ak[e] = ak[e] + to_f32<T>(ke[e]);
                }
            }
        }
    }
    uint4 oq, ok;
    T* oqe = reinterpret_cast<T*>(&oq);
    T* oke = reinterpret_cast<T*>(&ok);
#pragma unroll
    for (int e = 0; e < V; ++e) {
        // separate multiply after the sum: no contraction into an fma
        const float mq = __fmul_rn(aq[e], sh.inv_gsize);
        const float mk = __fmul_rn(ak[e], sh.inv_gsize);
        oqe[e] = from_f32_rne<T>(mq);
        oke[e] = from_f32_rne<T>(mk);
    }
    const int64_t o = ((int64_t)g * sh.np + tp) * D + slice * V;
    *reinterpret_cast<uint4*>(qg + o) = oq;
    *reinterpret_cast<uint4*>(kg + o) = ok;
}

// ---------------------------------------------------------------------------
// a2: per-(row, key block) max and per-(row, key chunk) (max, sum)
// One 256-thread workgroup per (128-row band, key chunk c, group g): it
// takes the strided rows R0 .. R0+127, wave w rows R0+32w..+31, against key
// tiles [c est_kc, (c+1) est_kc) of the causal range (chunks past it exit at
// once).  Only the wave's diagonal key tile needs the causal mask.  The
// per-(row, key block) maxima go to the current band group's rbm region:
// lower-triangular pairs (m, n) at tri_index(m, n) - tri_base, tri_count
// pairs per proxy group.
// ---------------------------------------------------------------------------
template <typename T, int D, int BP>
__device__ __forceinline__ void est_rowmax_body(const Shape& sh, const T* __restrict__ qg,
                                                const T* __restrict__ kg,
                                                float* __restrict__ rbm,
                                                float2* __restrict__ rowpart, int R0, int c, int g,
                                                int64_t tri_base, int64_t tri_count) {
    typedef typename OperandOf<T>::type Op;
    typedef StepCopy<T, D> Copy;
    constexpr int KS = D / 16;
    __shared__ __attribute__((aligned(16))) T tile0[Copy::ELEMS];
    __shared__ __attribute__((aligned(16))) T tile1[Copy::ELEMS];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, lc = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int np = sh.np;
    const int kt_begin = c * sh.est_kc;                    // a multiple of 4: 128 keys
    const int last_row_tile = min(R0 + 127, np - 1) / 32;
    if (kt_begin > last_row_tile) return;   // the whole workgroup: no barrier skipped
    const int s0 = kt_begin / 2, s1 = min(last_row_tile, kt_begin + sh.est_kc - 1) / 2;
    const int row0 = R0 + 32 * w, row = row0 + lc;
    // the wave's steps end with its diagonal
    const int ws1 = row0 < np ? min(s1, (row0 + 31) / kStepKeys) : s0 - 1;
    const float scale2 = sh.scale2;

    const T* kbase = kg + (int64_t)g * np * D;
    Copy copy(kbase, D, np, s0, w, lane);
    copy.issue(s0, tile0);
    Op qf[KS];
    {
        const T* qrow = qg + ((int64_t)g * np + min(row, np - 1)) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = query_operand(load_frag<T>(qrow + 16 * ks + 8 * h));
    }
    LaneLines<T, D> lines(lc, h);

    // Block maxima of a step: NV values a lane, value v (of lane half h) of
    // block first + 2 v + h for b' <= 32 (the halves take two blocks), of the
    // step's one block for b' >= 64 (half 0 stores it).  They are stored
    // after the next step's barrier, so that a wait for copies never waits
    // for a store just issued.
    constexpr int NV = BP == 16 ? 2 : 1, BPS = BP <= 32 ? kStepKeys / BP : 1;
    const int mr = row / BP;
    float* rrow = rbm + ((int64_t)g * tri_count - tri_base + tri_index(mr, 0)) * BP + row % BP;
    const int nmax = row >= np || (BP >= 64 && h) ? -1 : mr;   // last block to store
    float pend[NV];
    int pend_n = -1;   // first block of the pending values
    auto flush = [&]() {
        if (pend_n < 0) return;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int n = BP <= 32 ? pend_n + 2 * v + h : pend_n;
            if (n <= nmax) rrow[(int64_t)n * BP] = pend[v];
        }
        pend_n = -1;
    };

    // reference m (scaled, log2 units) and sum l of the running sum
    float m = kNegInf, neg = 0.f, l = 0.f, bm = kNegInf;
    auto step = [&](int st, T* cur, T* next) {
        lines.renew();
        wait_copies();      // tile st has landed ...
        __syncthreads();    // ... for every wave, and all are done with st - 1
        flush();
        if (st < s1) copy.issue(st + 1, next);
        if (st > ws1) return;
        f32x16 acc[2];
        const int k0 = st * kStepKeys;
        step_scores<T, D>(acc, cur, lines, qf, k0 + 32 > row0 + 31);
        if (k0 + kStepKeys - 1 > row0) step_mask(acc, row - k0, h);
        // raw maxima (the scale is positive, so it commutes with max)
        const float a0 = max8(acc[0], 0), a1 = max8(acc[0], 8);
        const float b0 = max8(acc[1], 0), b1 = max8(acc[1], 8);
        const float ta = fmaxf(a0, a1), tb = fmaxf(b0, b1), tm = fmaxf(ta, tb) * scale2;
        if (__builtin_amdgcn_ballot_w64(tm > m + kSumSlack)) {
            // a lane half can have all of its keys masked so far (m = -inf):
            // it then adds exp2(-inf) = 0 and keeps l = 0
            const float mn = fmaxf(m, tm);
            l *= m == kNegInf ? 0.f : fast_exp2(m - mn);
            m = mn;
            neg = m == kNegInf ? 0.f : -m;
        }
        l += step_sum(acc, scale2, neg);
        if constexpr (BP == 16) {   // slots r < 8 and r >= 8 of a tile are two blocks
            pend[0] = halves_max2(a0, a1) * scale2;
            pend[1] = halves_max2(b0, b1) * scale2;
            pend_n = 4 * st;
        } else if constexpr (BP == 32) {
            pend[0] = halves_max2(ta, tb) * scale2;
            pend_n = 2 * st;
        } else {
            const float sm = halves_max(tm);
            constexpr int SPB = BP / kStepKeys;   // steps per block
            bm = SPB == 1 || st % SPB == 0 ? sm : fmaxf(bm, sm);
            if (SPB == 1 || st % SPB == SPB - 1 || st == ws1) {
                pend[0] = bm;
                pend_n = st / SPB;
            }
        }
    };
    for (int st = s0; st <= s1; st += 2) {
        step(st, tile0, tile1);
        if (st < s1) step(st + 1, tile1, tile0);
    }
    flush();
    const float mo = swap_halves(m), lo = swap_halves(l);
    const float mm = fmaxf(m, mo);
    if (h == 0 && row < np) {
        // a half with m = -inf has l = 0; a row with no visible key in this
        // chunk writes (-inf, 0)
        const float ll = (m == kNegInf ? 0.f : l * fast_exp2(m - mm)) +
                         (mo == kNegInf ? 0.f : lo * fast_exp2(mo - mm));
        rowpart[((int64_t)g * sh.est_nc + c) * np + row] = make_float2(mm, ll);
    }
}

// ---------------------------------------------------------------------------
// a3: row normalisers and the block max-pool in the log domain.
// One 256-thread workgroup per (block row m, group g).
// ---------------------------------------------------------------------------

// Maximum over groups of W consecutive lanes (W = 4 .. 32), in every lane.
template <int W>
__device__ __forceinline__ float lanes_max(float v) {
    auto dpp = [](float x, auto ctrl) {
        const int i = __float_as_int(x);
        return __int_as_float(__builtin_amdgcn_update_dpp(i, i, decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0xB1>()));                        // quad_perm 1 0 3 2
    v = fmaxf(v, dpp(v, std::integral_constant<int, 0x4E>()));                        // quad_perm 2 3 0 1
    if constexpr (W >= 8) v = fmaxf(v, dpp(v, std::integral_constant<int, 0x141>())); // row_half_mirror
    if constexpr (W >= 16) v = fmaxf(v, dpp(v, std::integral_constant<int, 0x140>())); // row_mirror
    if constexpr (W >= 32) v = fmaxf(v, __shfl_xor(v, 16));
    return v;
}

template <int BP>
__device__ __forceinline__ void est_reduce_body(const Shape& sh, const float* __restrict__ rbm,
                                                const float2* __restrict__ rowpart,
                                                float* __restrict__ logA, int m, int g,
                                                int64_t tri_base, int64_t tri_count) {
    __shared__ __attribute__((aligned(16))) float L[BP];
    const int tid = threadIdx.x;
    const int r0 = m * BP;
    const int nr = min(BP, sh.np - r0);
    // the block's rows lie in one 128-row band of est_rowmax (BP divides
    // 128), which wrote chunks 0 .. nck-1 for them
    const int nck = (min((r0 / 128) * 128 + 127, sh.np - 1) / 32) / sh.est_kc + 1;
    // the chunk pairs are read kChunkBatch at a time, all in flight together
    // (a batch past the last chunk re-reads it: the max is unchanged and the
    // sum skips it); the sum runs over the chunks in increasing order
    constexpr int kChunkBatch = 8;
    for (int j = tid; j < BP; j += 256) {
        float v = 0.f;
        if (j < nr) {
            const float2* pp = rowpart + (int64_t)g * sh.est_nc * sh.np + r0 + j;
            float mx = kNegInf;
            for (int c0 = 0; c0 < nck; c0 += kChunkBatch) {
                float xs[kChunkBatch];
#pragma unroll
                for (int u = 0; u < kChunkBatch; ++u)
                    xs[u] = pp[(int64_t)min(c0 + u, nck - 1) * sh.np].x;
#pragma unroll
                for (int u = 0; u < kChunkBatch; ++u) mx = fmaxf(mx, xs[u]);
            }
            // mx is finite: key 0 (chunk 0) is visible to every row
            float sum = 0.f;
            for (int c0 = 0; c0 < nck; c0 += kChunkBatch) {
                float2 xs[kChunkBatch];
#pragma unroll
                for (int u = 0; u < kChunkBatch; ++u)
                    xs[u] = pp[(int64_t)min(c0 + u, nck - 1) * sh.np];
#pragma unroll
                for (int u = 0; u < kChunkBatch; ++u) {
                    // a select, not a branch, so that both halves of the
                    // pair are loaded with the one 8-byte load
                    const bool use = c0 + u < nck && xs[u].x != kNegInf;
                    sum = use ? fmaf(xs[u].y, fast_exp2(xs[u].x - mx), sum) : sum;
                }
            }
            v = mx + log2f(sum);
        }
        L[j] = v;
    }
    __syncthreads();
    const float* base = rbm + ((int64_t)g * tri_count + tri_index(m, 0) - tri_base) * BP;
    float* out = logA + ((int64_t)g * sh.mq + m) * sh.mq;
    if (nr == BP && sh.mq > 256) {
        // Bound by its loads.  A wave takes 64 blocks at a time, G = BP / 4
        // lanes to a block: its loads are whole contiguous KiB, kLoads of them
        // in flight.  A lane keeps the maximum of the blocks of load lane % G.
        // One lane to a block, below, reads 16 bytes of 64 lines at a time:
        // estimate call 128K 969 -> 959 us, 50K stride 2 913 -> 905 us, 64K 456
        // -> 452 us.  Up to 256 blocks (64 for each wave) there is one pass
        // either way, and this one was up to 0.6 % slower (8K, 16K).
        constexpr int G = BP / 4, PER = 64 / G, kLoads = G < 8 ? G : 8;
        const int lane = tid & 63, sub = lane % G, grp = lane / G;
        const f32x4 lr = *reinterpret_cast<const f32x4*>(L + 4 * sub);
        for (int n0 = tid - lane; n0 < sh.mq; n0 += 256) {
            const int n = n0 + sub * PER + grp;
            float v = kNegInf;
            if (n0 <= m) {
                for (int u0 = 0; u0 < G; u0 += kLoads) {
                    f32x4 x[kLoads];
#pragma unroll
                    for (int u = 0; u < kLoads; ++u)
                        x[u] = *reinterpret_cast<const f32x4*>(
                            base + (int64_t)min(n0 + (u0 + u) * PER + grp, m) * BP + 4 * sub);
#pragma unroll
                    for (int u = 0; u < kLoads; ++u) {
                        const float t = lanes_max<G>(fmaxf(fmaxf(x[u][0] - lr[0], x[u][1] - lr[1]),
                                                           fmaxf(x[u][2] - lr[2], x[u][3] - lr[3])));
                        v = sub == u0 + u ? t : v;
                    }
                }
                v = n <= m ? v * kLn2 : kNegInf;
            }
            if (n < sh.mq) out[n] = v;
        }
        return;
    }
    for (int n = tid; n < sh.mq; n += 256) {
        float v = kNegInf;
        if (n <= m) {
            const float* p = base + (int64_t)n * BP;
            if (nr == BP) {
#pragma unroll
                for (int j = 0; j < BP; j += 4) {
                    const f32x4 x = *reinterpret_cast<const f32x4*>(p + j);
                    v = fmaxf(v, fmaxf(fmaxf(x[0] - L[j], x[1] - L[j + 1]),
                                       fmaxf(x[2] - L[j + 2], x[3] - L[j + 3])));
                }
            } else {
                for (int j = 0; j < nr; ++j) v = fmaxf(v, p[j] - L[j]);
            }
            v *= kLn2;
        }
        out[n] = v;
    }
}

// ---------------------------------------------------------------------------
// a4: last-block mass, one pass over the keys.
// mass_block: one 256-thread workgroup per (key chunk c, head i); wave w
//   takes last-block rows 32w..32w+31 (b = 64: waves 2 and 3 only help to
//   stage the key tiles).  For every (row, key block) of its key chunk: the
//   block's largest scaled logit m and the sum of exp2(logit - m) over the
//   block's visible keys, written to part[i][row][block] (float2).
// mass_norm, mass_sum: each row's log2-sum-exp over its visible blocks, then
//   mass[i][n] = sum over rows of s * exp2(m - L) in a fixed order.
// ---------------------------------------------------------------------------
template <typename T, int D, int B>
__device__ __forceinline__ void mass_block_body(const Shape& sh, const T* __restrict__ q,
                                                const T* __restrict__ k,
                                                float2* __restrict__ part, int c, int i) {
    typedef typename OperandOf<T>::type Op;
    typedef StepCopy<T, D> Copy;
    static_assert(B <= 128, "at most 4 waves of 32 last-block rows");
    constexpr int SPB = B / kStepKeys;   // steps per block
    __shared__ __attribute__((aligned(16))) T tile0[Copy::ELEMS];
    __shared__ __attribute__((aligned(16))) T tile1[Copy::ELEMS];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, lc = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kvh = i / sh.rep;
    const int n = sh.n;
    const int nrows = min(B, n), t0 = n - nrows;
    const int rl = 32 * w + lc, t = t0 + rl;
    const bool wave_on = 32 * w < nrows;
    const int wave_first_t = t0 + 32 * w;
    const int wave_last_t = t0 + min(32 * w + 31, nrows - 1);
    const int key0 = c * sh.mass_chunk, key1 = min(key0 + sh.mass_chunk, n);
    const int s0 = key0 / kStepKeys, s1 = (key1 - 1) / kStepKeys;

    Copy copy(k + (int64_t)kvh * sh.kv_head, sh.kv_tok, n, s0, w, lane);
    copy.issue(s0, tile0);
    Op qf[D / 16];
    {
        const T* qrow = q + (int64_t)min(t, n - 1) * sh.q_tok + (int64_t)i * sh.q_head;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[ks] = query_operand(load_frag<T>(qrow + 16 * ks + 8 * h));
    }
    LaneLines<T, D> lines(lc, h);
    float2* prow = part + ((int64_t)i * B + rl) * sh.mq;
    float2 pend = make_float2(0.f, 0.f);
    int pend_n = -1;   // block of the pending pair (stored after the next barrier)
    auto flush = [&]() {
        if (pend_n < 0) return;
        if (wave_on && h == 0 && rl < nrows) prow[pend_n] = pend;
        pend_n = -1;
    };
    // the block's reference m (both halves of a row share it) and this lane's
    // sum
    float m = kNegInf, neg = 0.f, l = 0.f;
    auto step = [&](int st, T* cur, T* next) {
        lines.renew();
        wait_copies();      // tile st has landed ...
        __syncthreads();    // ... for every wave, and all are done with st - 1
        flush();
        if (st < s1) copy.issue(st + 1, next);
        if (!wave_on) return;
        f32x16 acc[2];
        const int k0 = st * kStepKeys;
        step_scores<T, D>(acc, cur, lines, qf, k0 + 32 > wave_last_t);
        // only steps reaching past the wave's first row need the causal mask
        if (k0 + kStepKeys - 1 > wave_first_t) step_mask(acc, t - k0, h);
        const float tm = halves_max(fmaxf(fmaxf(max8(acc[0], 0), max8(acc[0], 8)),
                                          fmaxf(max8(acc[1], 0), max8(acc[1], 8)))) * sh.scale2;
        if (SPB == 1 || st % SPB == 0) {   // a new block
            m = tm;
            neg = m == kNegInf ? 0.f : -m;
            l = 0.f;
        } else if (__builtin_amdgcn_ballot_w64(tm > m + kSumSlack)) {
            const float mn = fmaxf(m, tm);
            l *= m == kNegInf ? 0.f : fast_exp2(m - mn);
            m = mn;
            neg = m == kNegInf ? 0.f : -m;
        }
        l += step_sum(acc, sh.scale2, neg);
        if (SPB == 1 || st % SPB == SPB - 1 || st == s1) {
            pend = make_float2(m, halves_sum(l));
            pend_n = st / SPB;
        }
    };
    for (int st = s0; st <= s1; st += 2) {
        step(st, tile0, tile1);
        if (st < s1) step(st + 1, tile1, tile0);
    }
    flush();
}

// Row normalisers: W lanes per last-block row, 256 / W rows per 256-thread
// workgroup (`rg`: the workgroup's index among the head's): the row's
// log2-sum-exp over its visible blocks n <= t / b (block n holds key n b <= t,
// so every one of them was written).  A wave per row, or W = 8 up to 8 blocks:
// the workgroups share a launch with est_rowmax, whose tiles let only two to
// five of them on a CU, and layers of many heads have thousands.  Estimate
// call of 128 tokens, 512/64 heads, d 128 b 128, 64 lanes a row -> 8: fp32 72.9
// -> 35.7 us, bf16 41.5 -> 20.6 (with the smaller tiles of 32-key steps 63.6 and
// 37.3); 8/2 heads and longer calls as fast either way.  The sums' order is the
// same: lanes past the last block add 0.
constexpr int kNormShortBlocks = 8;

template <int W>
__device__ __forceinline__ void mass_norm_body(const Shape& sh, const float2* __restrict__ part,
                                               float* __restrict__ lnorm, int i, int rg) {
    const int sub = threadIdx.x % W;
    const int b = sh.b, mq = sh.mq;
    const int nrows = min(b, sh.n), t0 = sh.n - nrows;
    const int r = rg * (256 / W) + threadIdx.x / W;
    if (r >= nrows) return;   // whole rows; no barrier follows
    const int nmax = (t0 + r) / b;
    const float2* pr = part + ((int64_t)i * b + r) * mq;
    // a lane's blocks nb = sub, sub + W, ... in increasing order, read
    // kNormBatch at a time (all in flight together); selects, not branches,
    // so that each pair is one 8-byte load
    constexpr int kNormBatch = W == 64 ? 4 : 1;
    float m = kNegInf, s = 0.f;
    for (int nb0 = sub; nb0 <= nmax; nb0 += W * kNormBatch) {
        float2 xs[kNormBatch];
#pragma unroll
        for (int u = 0; u < kNormBatch; ++u) {
            const int nb = nb0 + W * u;
            xs[u] = pr[min(nb, nmax)];
        }
#pragma unroll
        for (int u = 0; u < kNormBatch; ++u) {
            const float2 x = xs[u];
            const bool use = nb0 + W * u <= nmax && x.x != kNegInf;
            const float mn = fmaxf(m, x.x);
            const float sn = (m == kNegInf ? 0.f : s * fast_exp2(m - mn)) + x.y * fast_exp2(x.x - mn);
            s = use ? sn : s;
            m = use ? mn : m;
        }
    }
    float M = m;   // finite in the end: block 0 is visible to every row
#pragma unroll
    for (int o = W / 2; o >= 1; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
    float sv = m == kNegInf ? 0.f : s * fast_exp2(m - M);
#pragma unroll
    for (int o = W / 2; o >= 1; o >>= 1) sv += __shfl_xor(sv, o);
    if (sub == 0) lnorm[(int64_t)i * b + r] = M + log2f(sv);
}

// Block masses: 64 blocks per 256-thread workgroup (`chunk`), one per lane.
// The fixed-order sum: partial p (p = 0..15) adds rows p, p + 16, ... in
// increasing order (wave w computes partials w, w + 4, w + 8, w + 12), then
// the 16 partials are added in order.
constexpr int kMassPartials = 16;

__device__ __forceinline__ void mass_sum_body(const Shape& sh, const float2* __restrict__ part,
                                              const float* __restrict__ lnorm,
                                              float* __restrict__ mass, int i, int chunk) {
    __shared__ float L[128];
    __shared__ float ps[kMassPartials][64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int b = sh.b, mq = sh.mq;
    const int nrows = min(b, sh.n), t0 = sh.n - nrows;
    for (int r = tid; r < nrows; r += 256) L[r] = lnorm[(int64_t)i * b + r];
    __syncthreads();
    const float2* base = part + (int64_t)i * b * mq;
    const int nb = chunk * 64 + lane;
    // a partial's rows (at most 128 / kMassPartials) are read together, all
    // in flight at once, then accumulated (one fma each) in increasing order;
    // an invisible block or a row past the last reads as (-inf, 0) and is
    // skipped (a select, not a branch, so that each pair is one 8-byte load)
    constexpr int kRowsPerPartial = 128 / kMassPartials;
#pragma unroll
    for (int pp = 0; pp < kMassPartials / 4; ++pp) {
        const int p = w + 4 * pp;
        float2 xs[kRowsPerPartial];
#pragma unroll
        for (int u = 0; u < kRowsPerPartial; ++u) {
            const int r = p + kMassPartials * u;
            xs[u] = (nb < mq && r < nrows && nb * b <= t0 + r) ? base[(int64_t)r * mq + nb]
                                                              : make_float2(kNegInf, 0.f);
        }
        float acc = 0.f;
#pragma unroll
        for (int u = 0; u < kRowsPerPartial; ++u) {
            const int r = min(p + kMassPartials * u, nrows - 1);
            acc = xs[u].x != kNegInf ? fmaf(xs[u].y, fast_exp2(xs[u].x - L[r]), acc) : acc;
        }
        ps[p][lane] = acc;
    }
    __syncthreads();
    if (w == 0 && nb < mq) {
        float sum = 0.f;
#pragma unroll
        for (int p = 0; p < kMassPartials; ++p) sum += ps[p][lane];
        mass[(int64_t)i * mq + nb] = sum;
    }
}

// ---------------------------------------------------------------------------
// The three fused launches (1-D grids of 256-thread workgroups; the
// workgroups of the longer role come first).
// ---------------------------------------------------------------------------
struct EstGrid {
    int pool;      // pooling workgroups: G x pool_per
    int pool_per;  // per group
    int mblock;    // mass_block workgroups: nchunks x Hq
    int rowmax;    // est_rowmax workgroups: nbx x est_nc x G (of the band group)
    int nbx;       // 128-row bands of est_rowmax in the band group
    int xb1;       // one past the group's last band (bands run longest first)
    int norm;      // mass_norm workgroups: Hq x norm_per (first group only)
    int norm_per;  // per head
    int reduce;    // est_reduce workgroups: the group's block rows x G
    int m0, nm;    // the group's block rows [m0, m0 + nm)
    int msum;      // mass_sum workgroups: Hq x ceil(Nk / 64) (first group only)
    int msum_per;  // per head
    int64_t tri_base;   // tri_index(m0, 0)
    int64_t tri_count;  // lower-triangular pairs of the group's block rows
};

template <typename T, int D, int B>
__global__ __launch_bounds__(256, 2) void est_stage1_kernel(Shape sh, EstGrid eg,
                                                            const T* __restrict__ q,
                                                            const T* __restrict__ k,
                                                            T* __restrict__ qg, T* __restrict__ kg,
                                                            float2* __restrict__ part) {
    const int j = blockIdx.x;
    if (j < eg.mblock) {
        mass_block_body<T, D, B>(sh, q, k, part, j % sh.nchunks, j / sh.nchunks);
        return;
    }
    const int jp = j - eg.mblock;
    pool_body<T, D>(sh, q, k, qg, kg, jp / eg.pool_per, jp % eg.pool_per);
}

template <typename T, int D, int BP>
__global__ __launch_bounds__(256, 2) void est_stage2_kernel(Shape sh, EstGrid eg,
                                                            const T* __restrict__ qg,
                                                            const T* __restrict__ kg,
                                                            float* __restrict__ rbm,
                                                            float2* __restrict__ rowpart,
                                                            const float2* __restrict__ part,
                                                            float* __restrict__ lnorm) {
    const int j = blockIdx.x;
    if (j < eg.rowmax) {
        const int bx = j % eg.nbx, c = (j / eg.nbx) % sh.est_nc, g = j / (eg.nbx * sh.est_nc);
        est_rowmax_body<T, D, BP>(sh, qg, kg, rbm, rowpart, (eg.xb1 - 1 - bx) * 128, c, g,
                                  eg.tri_base, eg.tri_count);
        return;
    }
    const int jn = j - eg.rowmax;
    if (sh.mq <= kNormShortBlocks)
        mass_norm_body<8>(sh, part, lnorm, jn / eg.norm_per, jn % eg.norm_per);
    else
        mass_norm_body<64>(sh, part, lnorm, jn / eg.norm_per, jn % eg.norm_per);
}

template <int BP>
__global__ __launch_bounds__(256) void est_stage3_kernel(Shape sh, EstGrid eg,
                                                         const float* __restrict__ rbm,
                                                         const float2* __restrict__ rowpart,
                                                         float* __restrict__ logA,
                                                         const float2* __restrict__ part,
                                                         const float* __restrict__ lnorm,
                                                         float* __restrict__ mass) {
    const int j = blockIdx.x;
    if (j < eg.reduce) {
        est_reduce_body<BP>(sh, rbm, rowpart, logA, eg.m0 + j % eg.nm, j / eg.nm, eg.tri_base,
                            eg.tri_count);
        return;
    }
    const int jm = j - eg.reduce;
    mass_sum_body(sh, part, lnorm, mass, jm / eg.msum_per, jm % eg.msum_per);
}

// ---------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------
static EstGrid est_grid(const Shape& sh) {
    EstGrid e{};
    constexpr int kVec = 16;   // bytes per pooled slice
    const int esz = sh.dtype == 0 ? 2 : 4;
    const int slices = sh.d * esz / kVec;
    e.pool_per = (int)(((int64_t)sh.np * slices + 255) / 256);
    e.pool = sh.g * e.pool_per;
    e.mblock = sh.nchunks * sh.hq;
    const int norm_rows = 256 / (sh.mq <= kNormShortBlocks ? 8 : 64);   // of a workgroup
    e.norm_per = (std::min(sh.b, sh.n) + norm_rows - 1) / norm_rows;
    e.norm = sh.hq * e.norm_per;
    e.msum_per = (sh.mq + 63) / 64;
    e.msum = sh.hq * e.msum_per;
    return e;
}

// Band group k of est_rowmax / est_reduce (see rbm_groups): bands [xb0, xb1)
// of 128 strided rows, block rows [m0, m1).
static void set_group(const Shape& sh, const RbmGroup& gr, bool first, EstGrid* e) {
    const int rows_per_band = 128 / sh.bp;   // block rows per 128-row band
    e->xb1 = gr.xb1;
    e->nbx = gr.xb1 - gr.xb0;
    e->rowmax = e->nbx * sh.est_nc * sh.g;
    e->m0 = gr.xb0 * rows_per_band;
    const int m1 = std::min(gr.xb1 * rows_per_band, sh.mq);
    e->nm = m1 - e->m0;
    e->reduce = e->nm * sh.g;
    e->tri_base = (int64_t)e->m0 * (e->m0 + 1) / 2;
    e->tri_count = (int64_t)m1 * (m1 + 1) / 2 - e->tri_base;
    if (!first) e->norm = e->msum = 0;
}

template <typename T, int D, int B, int BP>
static hipError_t est_t(const Shape& sh, const void* q, const void* k, const EstWs& w,
                        float* logA, float* mass, hipStream_t st) {
    EstGrid eg = est_grid(sh);
    hipLaunchKernelGGL((est_stage1_kernel<T, D, B>), dim3(eg.mblock + eg.pool), dim3(256), 0, st, sh,
                       eg, (const T*)q, (const T*)k, (T*)w.qg, (T*)w.kg, w.part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // est_rowmax writes and est_reduce reads the per-(row, block) maxima one
    // band group at a time, so that their region stays bounded (one group,
    // the whole range, unless it would exceed kRbmMaxBytes); the mass
    // stages ride along with the first group
    const int ngroups = rbm_groups(sh, nullptr);
    for (int k = 0; k < ngroups; ++k) {
        RbmGroup gr;
        rbm_group(sh, k, &gr);
        set_group(sh, gr, k == 0, &eg);
        hipLaunchKernelGGL((est_stage2_kernel<T, D, BP>), dim3(eg.rowmax + eg.norm), dim3(256), 0,
                           st, sh, eg, (const T*)w.qg, (const T*)w.kg, w.rbm, w.rowpart,
                           (const float2*)w.part, w.lnorm);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((est_stage3_kernel<BP>), dim3(eg.reduce + eg.msum), dim3(256), 0, st, sh,
                           eg, (const float*)w.rbm, (const float2*)w.rowpart, logA,
                           (const float2*)w.part, (const float*)w.lnorm, mass);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T, int D, int B>
static hipError_t est_bp(const Shape& sh, const void* q, const void* k, const EstWs& w,
                         float* logA, float* mass, hipStream_t st) {
    switch (sh.bp) {
        case 16: return est_t<T, D, B, 16>(sh, q, k, w, logA, mass, st);
        case 32: return est_t<T, D, B, 32>(sh, q, k, w, logA, mass, st);
        case 64: return est_t<T, D, B, 64>(sh, q, k, w, logA, mass, st);
        case 128: return est_t<T, D, B, 128>(sh, q, k, w, logA, mass, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_estimate(const Shape& sh, const void* q, const void* k, const EstWs& w,
                           float* logA, float* mass, hipStream_t st) {
    if (sh.dtype == 0) {
        if (sh.d == 64) return sh.b == 64 ? est_bp<bf16, 64, 64>(sh, q, k, w, logA, mass, st)
                                          : est_bp<bf16, 64, 128>(sh, q, k, w, logA, mass, st);
        return sh.b == 64 ? est_bp<bf16, 128, 64>(sh, q, k, w, logA, mass, st)
                          : est_bp<bf16, 128, 128>(sh, q, k, w, logA, mass, st);
    }
    if (sh.d == 64) return sh.b == 64 ? est_bp<float, 64, 64>(sh, q, k, w, logA, mass, st)
                                      : est_bp<float, 64, 128>(sh, q, k, w, logA, mass, st);
    return sh.b == 64 ? est_bp<float, 128, 64>(sh, q, k, w, logA, mass, st)
                      : est_bp<float, 128, 128>(sh, q, k, w, logA, mass, st);
}

}  // namespace pa
