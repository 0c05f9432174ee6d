// Causal block-sparse attention over the selected blocks (Sec. 3.2, last
// paragraph) and its dense baseline (every causal block).
//
// Work item = (query head i, query block m): b query rows, one wave per 32
// rows.  The item walks its list of key blocks in sub-blocks of 64 or 32
// keys (see sub_keys); for each sub-block it computes
//   S^T = K Q^T            (32x32x16 bf16 MFMA; K from LDS, Q in registers)
//   online softmax          (lane-local per query + one half-wave exchange)
//   O^T += V^T P^T          (P^T straight from the S^T accumulators)
// Each lane owns one query column of every tile, so the probabilities in
// S^T's accumulators are already laid out as the B operand of the PV
// product: a 32-key tile's 16 accumulator slots of lane half h cover keys
// 8(r/4) + 4h + r%4, and the V^T operand is read in that key order.
//
// A pre-pass re-blocks K and V once per call into
//   kvb[h][n][sub] = { K tile, V^T tile }     (KT keys each, see line_pos)
// with the keys of V^T permuted (bits 2 and 3 of the offset in each 32-key
// tile swapped), so that every sub-block is one contiguous chunk (spread over
// all HBM channels whatever KV head is being read), the 8 keys a lane needs
// for one PV step are contiguous, and rows past N are zero.
//
// Pipeline (one barrier per step j; two workgroups share a CU):
//   - sub-tiles are copied global -> LDS with buffer loads (no staging
//     registers); K and V^T have separate double buffers, K one step ahead:
//     during step j the copies of K(j+2) and V(j+1) run while the wave reads
//     K(j+1) and V(j);
//   - bf16: the scores of step j+1 (MFMA), then PV of step j, run as one
//     explicit software pipeline in which every LDS fragment read is issued
//     kReadLead MFMAs ahead of its use and step j+1's probabilities (VALU)
//     are formed beside the PV MFMAs; the reference of the online softmax is
//     checked after the fact, at the start of the next step;
//   - fp32: the same MFMA order with three bf16 terms per operand (Split3);
//     a fragment is split beside the MFMAs of the one before, and a step's
//     probabilities are formed beside the next step's scores.
#include <algorithm>
#include <mutex>
#include <vector>

#include "common.h"
#include "internal.h"
#include "work_order.h"

namespace pa {

__device__ __forceinline__ int swap_bits23(int x) {
    return (x & ~12) | ((x & 4) << 1) | ((x & 8) >> 1);
}

// Keys per sub-block (one step of the attention loop).  A workgroup keeps
// two K and two V^T tiles in LDS.  At d = 128, b = 64 there are two waves to a
// workgroup, and with 64-key tiles (bf16 64 KiB, fp32 128 KiB) a CU's LDS
// holds two of them (fp32: one), one wave per SIMD (half); 32-key tiles give
// twice that (sparse, 32/8 heads: bf16 12K 516 -> 434 us, fp32 8K 1561 -> 985
// us).  bf16 at d = 64: 64-key tiles leave room for two waves per SIMD anyway,
// and 32-key ones were slower at two, three and four waves (20K, b = 64: 579
// against 607, 608, 615 us; b = 128: 534 against 560-570).  fp32 at d = 64, b =
// 128: as fast either way, but 64-key steps spill registers.  fp32 with d = b:
// 32-key steps were slower (d 64 dense 5K 347 -> 382 us, d 128 8K 917 -> 1009).
template <typename T, int D, int B>
constexpr int sub_keys() {
    return (D == 128 && B == 64) || (sizeof(T) == 4 && D == 64 && B == 128) ? 32 : 64;
}

// Tile layout of a sub-block (in the copy and in LDS alike, so that a tile
// moves to LDS as one contiguous run): lines of D elements (see line_pos).
// K: line = key.  V^T: row d's KT keys are segment (d / 32) % R of line
// 32 (d / 32 / R) + d % 32, R = D / KT rows to a line; so lane lc of a wave
// finds every fragment of both tiles in lines lc, lc + 32, ...

// ---------------------------------------------------------------------------
// K, V -> kvb.  grid (Mq, Hkv), 256 threads.  Rows >= N are zero.  Also
// zeroes the attention work-queue counters.
// ---------------------------------------------------------------------------

template <typename T, int D, int B>
__global__ __launch_bounds__(256) void kv_block_kernel(Shape sh, const T* __restrict__ k,
                                                       const T* __restrict__ v,
                                                       T* __restrict__ kvb,
                                                       int* __restrict__ queue) {
    static_assert(kNumXcd * kQueueStride <= 256, "one thread per queue word");
    if (queue && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kNumXcd * kQueueStride)
        queue[threadIdx.x] = 0;
    constexpr int V = Vec16<T>::n;
    constexpr int LDR = D + V;
    constexpr int KT = sub_keys<T, D, B>();
    constexpr int SUB = 2 * KT * D;
    __shared__ __attribute__((aligned(16))) T tile[B * LDR];
    const int blk = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const T* ksrc = k + (int64_t)h * sh.kv_head;
    const T* vsrc = v + (int64_t)h * sh.kv_head;
    T* dst = kvb + ((int64_t)h * sh.mq + blk) * (2 * B * D);
    for (int vi = tid; vi < B * D / V; vi += 256) {
        const int row = vi / (D / V), col = (vi % (D / V)) * V;
        const int tok = blk * B + row;
        u32x4 xk = zero_u32x4(), xv = zero_u32x4();
        if (tok < sh.n) {
            xk = *reinterpret_cast<const u32x4*>(ksrc + (int64_t)tok * sh.kv_tok + col);
            xv = *reinterpret_cast<const u32x4*>(vsrc + (int64_t)tok * sh.kv_tok + col);
        }
        // K rows go straight to their sub-block
        T* kd = dst + (row / KT) * SUB + line_pos<T, D>(row % KT, col);
        *reinterpret_cast<u32x4*>(kd) = xk;
        *reinterpret_cast<u32x4*>(tile + row * LDR + col) = xv;
    }
    __syncthreads();
    // V^T: row d of sub-block `sub` holds its KT keys in permuted order
    for (int ov = tid; ov < D * B / V; ov += 256) {
        const int sub = ov / (D * KT / V);
        const int rem = ov % (D * KT / V);
        const int d = rem / (KT / V), p0 = (rem % (KT / V)) * V;
        u32x4 x = zero_u32x4();
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int p = p0 + e;
            const int key = sub * KT + ((p & ~31) | swap_bits23(p & 31));
            put_elem<T>(x, e, tile[key * LDR + d]);
        }
        constexpr int R = D / KT;
        const int line = 32 * (d / 32 / R) + d % 32, elem = (d / 32 % R) * KT + p0;
        *reinterpret_cast<u32x4*>(dst + sub * SUB + KT * D + line_pos<T, D>(line, elem)) = x;
    }
}

// Clears the attention work-queue counters (a fill kernel rather than a
// memset, so that the sequence stays correct when a caller records it in a
// graph).
__global__ __launch_bounds__(256) void queue_reset_kernel(int* __restrict__ queue) {
    if (threadIdx.x < kNumXcd * kQueueStride) queue[threadIdx.x] = 0;
}

hipError_t launch_queue_reset(int* queue, hipStream_t st) {
    hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(256), 0, st, queue);
    return hipGetLastError();
}

// Scratch of the entry point that allocates nothing: the work-queue counters
// live in this file-scope device array, one copy per GPU, for the life of
// the process.  Host code never passes the array's name to a kernel (on the
// host it is only a stand-in for the symbol); it uses the device address
// that hipGetSymbolAddress returns, looked up once per device with that
// device current and kept in scratch_ptr[].
static __device__ __align__(256) int scratch[kScratchBytes / sizeof(int)];
static_assert(kQueueBytes <= kScratchBytes, "the work queues fit the scratch array");

constexpr int kMaxDevices = 64;
static std::mutex scratch_mu;
static int* scratch_ptr[kMaxDevices];

hipError_t scratch_address(int** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(scratch_mu);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        scratch_ptr[dev] = (int*)p;
    }
    *out = scratch_ptr[dev];
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// attention.  Persistent grid (one workgroup per resident slot), 2B threads (B/32
// waves), 2 workgroups per CU.
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ T cvt_p(float p);
template <> __device__ __forceinline__ bf16 cvt_p<bf16>(float p) { return (bf16)p; }
template <> __device__ __forceinline__ float cvt_p<float>(float p) { return p; }

// Slack (log2 units) by which a row max may exceed the running reference max
// before the accumulators are rescaled.
constexpr float kRescaleSlack = 8.f;

template <typename T, int D, int B>
struct AttnCfg {
    static constexpr int V = Vec16<T>::n;
    static constexpr int NTH = 2 * B;                  // B/32 waves
    static constexpr int KT = sub_keys<T, D, B>();      // keys per sub-block
    static constexpr int NSUB = B / KT;                // sub-blocks per block
    static constexpr int NT = KT / 32;                 // 32-key tiles per sub-block
    static constexpr int SUB = 2 * KT * D;             // elements of a kvb sub-block
    static constexpr int K_ELEMS = KT * D;             // K tile (swizzled rows)
    static constexpr int V_ELEMS = D * KT;             // V^T tile
    static constexpr int STAGE = K_ELEMS + V_ELEMS;
    // Waves per SIMD the LDS of one CU (160 KiB) leaves room for, capped at
    // 2: the kernel's register budget.  fp32 with d = b, and at d = 128, is
    // held to one wave per SIMD by LDS.
    static constexpr int LDS_BYTES = 2 * STAGE * (int)sizeof(T) + 16;
    // The same with G groups of waves to a workgroup (see attn_kernel).
    static constexpr int lds_bytes(int G) { return G * (LDS_BYTES + B * 8); }
    static constexpr int min_waves(int G) {
        const int n = (160 * 1024 / lds_bytes(G)) * (G * NTH / 64) / 4;
        return n < 1 ? 1 : (n > 2 ? 2 : n);
    }
    // Two groups fit a CU's LDS (all but fp32 at d = b = 128) and pay: bf16 at
    // d = b = 128 already keeps a CU's matrix pipes busy with one four-wave
    // workgroup's 32 rows a wave, and lists are short in 128-key blocks
    // (sparse 32 heads 512: 17.5 -> 19.9 us, 1K: 23.7 -> 26.2, 8 heads 4K: 43.8
    // -> 44.0 us; only dense 1K gained, 48.3 -> 39.4 us).
    static constexpr bool CAN_SPLIT = lds_bytes(2) <= 160 * 1024 && !(sizeof(T) == 2 && D == 128 && B == 128);
};

// Direct global -> LDS copy of one kvb sub-block (a K tile, then a V^T
// tile, both stored as they lie in LDS).  One buffer_load_dwordx4 ... lds
// moves 64 consecutive 16-byte slots (slot = lane); a tile's instructions are
// dealt to the waves round-robin.  The buffer descriptor spans exactly the
// sub-block (built in SGPRs per copy), so every instruction takes the same
// lane offset plus a constant, and the hardware range check keeps every read
// inside the sub-block.
template <typename T, int D, int KT, int NW>
struct SubTileDma {
    static constexpr int V = Vec16<T>::n;
    static constexpr int INS = KT * D / V / 64;        // wave instructions per tile
    static constexpr int J = INS / NW;                 // per wave
    static constexpr int TILE_BYTES = KT * D * (int)sizeof(T);
    static_assert(KT * D / V % (64 * NW) == 0, "whole wave instructions, the same for every wave");

    uint32_t off;   // byte offset of this lane's slot of the wave's first instruction
    int w;

    __device__ __forceinline__ SubTileDma(int w_, int lane) : off((w_ * 64 + lane) * 16), w(w_) {}
    __device__ __forceinline__ void issue(const T* sub, T* lds, int tile) const {
        // raw buffer, 32-bit dword format (CDNA descriptor word 3)
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<T*>(sub), 0, 2 * TILE_BYTES, 0x00020000);
#pragma unroll
        for (int j = 0; j < J; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                r, (__attribute__((address_space(3))) void*)(lds + (w + j * NW) * 64 * V), 16, off,
                tile * TILE_BYTES + j * NW * 1024, 0, 0);
    }
    __device__ __forceinline__ void issue_k(const T* sub, T* k_lds) const { issue(sub, k_lds, 0); }
    __device__ __forceinline__ void issue_v(const T* sub, T* v_lds) const { issue(sub, v_lds, 1); }
};

// The two K and two V^T tiles in LDS.  They are four separate variables so
// that each has an alias scope of its own: the compiler then sees that the
// reads of one slot do not depend on the copy in flight into another, and
// does not make them wait for it.
template <typename T>
struct LdsSlots {
    T* k0;
    T* k1;
    T* v0;
    T* v1;
    __device__ __forceinline__ T* k(int p) const { return p ? k1 : k0; }
    __device__ __forceinline__ T* v(int p) const { return p ? v1 : v0; }
};

// MFMAs between the LDS read of an operand fragment and the MFMA that uses it
// (bf16 attention loop).  With the probabilities formed in the PV segments,
// 3 is 0.3-0.7 % faster than 2 (8K to 128K, sparse and dense; 2 was the
// better lead while the QK segments carried the softmax).
constexpr int kReadLead = 3;
// Largest sum of one lane's probabilities in a step that certainly leaves the
// lazily rescaled reference in place: every bf16 probability is then at most
// 2^7, so its exponent is below log2(2^7 (1 + 2^-8)) < kRescaleSlack.
constexpr float kLazySum = 128.f;

// Causal / ragged mask of one sub-tile: keys past `lim` (offset of
// the last visible key inside the sub-tile) become -inf.  A key's offset is
// 32 kt + 8 (r/4) + (r%4) + 4 h; the compile-time part is compared with the
// per-lane limit lim - 4h.
template <int NT>
__device__ __forceinline__ void mask_tail(f32x16* s, int lim, int h) {
    const int lim_h = lim - 4 * h;
#pragma unroll
    for (int kt = 0; kt < NT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            s[kt][r] = (32 * kt + 8 * (r >> 2) + (r & 3) <= lim_h) ? s[kt][r] : kNegInf;
}

// Max of a lane's raw scores over the sub-tile, then over both wave halves
// (four independent chains instead of one serial one).
template <int NT>
__device__ __forceinline__ float tile_max(const f32x16* s) {
    float c[4] = {kNegInf, kNegInf, kNegInf, kNegInf};
#pragma unroll
    for (int kt = 0; kt < NT; ++kt)
#pragma unroll
        for (int r = 0; r < 16; r += 2) c[(r >> 1) & 3] = fmaxf(c[(r >> 1) & 3], fmaxf(s[kt][r], s[kt][r + 1]));
    return halves_max(fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3])));
}

// Sum of the bf16 probabilities a lane feeds to the PV product, two per
// v_dot2_f32_bf16 (the sum then matches the rounded P the MFMA consumes).
template <int NT>
__device__ __forceinline__ float prob_sum(const bf16x8 (*pf)[2]) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 one = {(__bf16)1.0f, (__bf16)1.0f};
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < NT; ++kt)
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bf16x2 pr = {pf[kt][e][2 * j], pf[kt][e][2 * j + 1]};
                acc[j] = __builtin_amdgcn_fdot2_f32_bf16(pr, one, acc[j], false);
            }
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Accumulators of group 1 on their way to group 0, through the tiles: register
// quad rg of wave w is a 1 KiB run, 16 bytes a lane, the quads of output tile
// dt at the end of array dt of the four that hold both groups' tiles (`slot`:
// group 0's).  At d = 128 that is group 1's tile alone.
template <typename T, int D, int B>
__device__ __forceinline__ f32x4* acc_quad(const LdsSlots<T>& slot, int w, int dt, int rg, int lane) {
    constexpr int RUNS = 2 * AttnCfg<T, D, B>::K_ELEMS * (int)sizeof(T) / 1024;   // per array
    constexpr int NEED = B / 32 * 4;
    static_assert(AttnCfg<T, D, B>::K_ELEMS == AttnCfg<T, D, B>::V_ELEMS, "equal tiles");
    static_assert(NEED <= (D == 128 ? RUNS / 2 : RUNS), "O fits the tiles");
    T* tiles = dt == 0 ? slot.k0 : dt == 1 ? slot.k1 : dt == 2 ? slot.v0 : slot.v1;
    return reinterpret_cast<f32x4*>(tiles) + (RUNS - NEED + w * 4 + rg) * 64 + lane;
}

// One work item: query block m of query head i.  Every wave of the
// workgroup calls it with the same (m, i); it starts and ends with no copy
// in flight, and the caller's barrier separates it from the previous item's
// LDS reads.  G = 2: the second group of waves (grp 1, with tiles of its own)
// walks the second half of the list, and group 0 joins the two.
template <typename T, int D, int B, bool DENSE, int G>
__device__ __forceinline__ void attn_one(const Shape& sh, const T* __restrict__ q,
                                         const T* __restrict__ kvb,
                                         const int* __restrict__ block_count,
                                         const int* __restrict__ block_index,
                                         T* __restrict__ out, float* __restrict__ lse,
                                         const int m, const int i,
                                         const LdsSlots<T>& slot, const int grp,
                                         float2* __restrict__ ml) {
    typedef AttnCfg<T, D, B> C;
    typedef typename FragOf<T>::type Frag;
    typedef SubTileDma<T, D, C::KT, C::NTH / 64> Dma;
    constexpr int NT = C::NT;
    constexpr int DT = D / 32;   // output tiles along d
    constexpr int KS = D / 16;   // k steps of Q K^T

    const int tid = threadIdx.x - grp * C::NTH, lane = tid & 63, w = tid >> 6, h = lane >> 5, lc = lane & 31;
    const int kvh = i / sh.rep;
    const int n_tok = sh.n;
    // counts and indices are clamped to the causal range, so malformed caller
    // lists give wrong values but never an out-of-bounds access
    const int cnt_all = DENSE ? (m + 1) : min(block_count[(int64_t)i * sh.mq + m], m + 1);
    // this group's entries of the list: [first, first + cnt), cnt <= per
    const int per = (cnt_all + G - 1) / G, first = grp * per;
    const int cnt = G == 1 ? cnt_all : min(max(cnt_all - first, 0), per);
    const int* list = DENSE ? nullptr : block_index + ((int64_t)i * sh.mq + m) * sh.mq + first;
    const int qtok = m * B + 32 * w + lc;
    const bool qvalid = qtok < n_tok;
    const int qlim = min(qtok, n_tok - 1);   // last key this row may see

    if (cnt_all <= 0) {   // the whole workgroup
        if (grp == 0 && qvalid) {
            T* orow = out + (int64_t)qtok * sh.o_tok + (int64_t)i * sh.o_head;
            // lane half h zeroes elements [h D/2, (h+1) D/2); a rolled loop,
            // so that no per-lane address stays live across work items
            u32x4* o4 = reinterpret_cast<u32x4*>(orow + h * (D / 2));
#pragma unroll 1
            for (int e = 0; e < D / 2 / Vec16<T>::n; ++e) o4[e] = zero_u32x4();
            if (lse && h == 0) lse[(int64_t)i * n_tok + qtok] = kNegInf;
        }
        return;
    }

    typedef typename OperandOf<T>::type Op;
    Op qf[KS];
    {
        const T* qrow = q + (int64_t)min(qtok, n_tok - 1) * sh.q_tok + (int64_t)i * sh.q_head;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = query_operand(load_frag<T>(qrow + 16 * ks + 8 * h));
    }

    const T* kvbase = kvb + (int64_t)kvh * sh.mq * (2 * B * D);
    // step j = sub-block (j % NSUB) of listed block (j / NSUB).  List entries
    // arrive 64 at a time, one per lane, through a vector load, and are picked
    // with v_readlane: no scalar-memory load in the loop, whose out-of-order
    // return would force every LDS wait to drain completely.
    int lst_base = -64, lst = 0;
    auto block_of = [&](int it) -> int {
        if (DENSE) return G == 1 ? it : min(first + it, m);
        const int c0 = it & ~63;
        if (c0 != lst_base) {
            lst_base = c0;
            lst = (c0 + lane < cnt) ? list[c0 + lane] : 0;
        }
        return min(max(__builtin_amdgcn_readlane(lst, it & 63), 0), m);
    };
    auto sub_src = [&](int nb, int sub) { return kvbase + (int64_t)nb * (2 * B * D) + sub * C::SUB; };
    auto needs_mask = [&](int nb) { return nb == m || (nb + 1) * B > n_tok; };
    // this lane's fragments of a K tile (key 32 kt + lc, elements 16 ks + 8 h
    // .. + 7) and of a V^T tile (row 32 dt + lc, the 8 keys of PV step (kt, e))
    LaneLines<T, D> lines(lc, h);
    auto kfrag = [&](const T* kb, int kt, int ks) { return lines.frag(kb + 32 * kt * D, 16 * ks); };
    auto vfrag = [&](const T* vb, int dt, int kt, int e) {
        constexpr int R = D / C::KT;
        return lines.frag(vb + 32 * (dt / R) * D, dt % R * C::KT + 32 * kt + 16 * e);
    };
    auto qk = [&](f32x16* acc, const T* kt_) {
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) {
            acc[kt] = zero16();
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) mma(acc[kt], key_operand(kfrag(kt_, kt, ks)), qf[ks]);
        }
    };

    float m_run = kNegInf, l_run = 0.f;
    f32x16 o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt] = zero16();

    // (a group without entries goes through the prologue on some block of the
    // causal range and drops what it finds)
    const int steps = cnt * C::NSUB;
    auto nb_of_step = [&](int j, int nb_prev) {
        return (j % C::NSUB == 0) ? block_of(j / C::NSUB) : nb_prev;
    };
    // prologue: K of steps 0 and 1, V of step 0; scores and max of step 0
    int nb0 = block_of(0);
    int nb1 = steps > 1 ? nb_of_step(1, nb0) : nb0;
    const Dma dma(w, lane);
    dma.issue_k(sub_src(nb0, 0), slot.k(0));
    dma.issue_v(sub_src(nb0, 0), slot.v(0));
    if (steps > 1) dma.issue_k(sub_src(nb1, 1 % C::NSUB), slot.k(1));
    wait_copies();
    __syncthreads();
    f32x16 s_cur[NT];
    qk(s_cur, slot.k(0));
    if (needs_mask(nb0)) mask_tail<NT>(s_cur, qlim - nb0 * B, h);
    float mx = tile_max<NT>(s_cur) * sh.scale2;

    // probabilities of the step the PV MFMAs consume next, from its scores
    Frag pf[NT][2];
    auto form_p = [&](const f32x16* s, float nm) {
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                pf[kt][r >> 3][r & 7] = cvt_p<T>(fast_exp2(fmaf(s[kt][r], sh.scale2, nm)));
    };
    // the reference moves only when some row's max exceeds it by more than
    // kRescaleSlack (probabilities stay < 2^8)
    auto rescale_to = [&](float mxs) {
        const float m_new = fmaxf(m_run, mxs);
        const float alpha = (m_run == kNegInf) ? 0.f : fast_exp2(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
        m_run = m_new;
    };
    // a row whose keys so far are all masked keeps m_run = -inf: its
    // probabilities are exp2(-inf) = 0
    auto neg_ref = [&]() { return (m_run == kNegInf) ? 0.f : -m_run; };
    if constexpr (sizeof(T) == 2) {
        // bf16: the first step's reference and probabilities here; later
        // steps form theirs in the PV segments of the step before
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleSlack)) rescale_to(mx);
        form_p(s_cur, neg_ref());
    }

    // One step.  `sc` holds the scores of step st, `sn` receives those
    // of step st+1 (two distinct register sets, used alternately, so the next
    // scores never wait for the current softmax to free its registers; bf16
    // keeps `sc` only for the step's rescale check).
    auto step = [&](f32x16* sc, f32x16* sn, int st) {
        lines.renew();
        if constexpr (sizeof(T) == 2) {
            // a masked sub-tile (the diagonal or a ragged end, rare): its
            // probabilities formed again from its masked scores
            if (st > 0 && needs_mask(nb0)) {
                mask_tail<NT>(sc, qlim - nb0 * B - (st % C::NSUB) * C::KT, h);
                form_p(sc, neg_ref());
            }
        }
        // K(st+1) and V(st) have landed; every wave is done with step st-1,
        // whose slots (K(st), V(st-1)) the next copies overwrite
        wait_copies();
        __syncthreads();
        int nb2 = nb1;
        if (st + 2 < steps) {
            nb2 = nb_of_step(st + 2, nb1);
            dma.issue_k(sub_src(nb2, (st + 2) % C::NSUB), slot.k(st & 1));
        }
        if (st + 1 < steps) dma.issue_v(sub_src(nb1, (st + 1) % C::NSUB), slot.v((st + 1) & 1));

        if constexpr (sizeof(T) == 2) {
            // Lazy rescaling checked after the fact.  The step's
            // probabilities were formed against the reference of the step
            // before (a masked sub-tile, rare, forms them again from its
            // masked scores).  A lane whose probabilities sum to at most
            // kLazySum holds none above it, so its row max exceeds the
            // reference by less than kRescaleSlack and the reference stays,
            // as the max itself would decide; otherwise (rare, and always on
            // overflow or while a row has no reference) the row max is taken
            // and, where the reference moves, the probabilities formed
            // again: the same decisions and values as taking the max first.
            float ps = prob_sum<NT>(pf);
            if (__builtin_amdgcn_ballot_w64(!(ps <= kLazySum) || m_run == kNegInf)) {
                const float mxs = tile_max<NT>(sc) * sh.scale2;
                if (__builtin_amdgcn_ballot_w64(mxs > m_run + kRescaleSlack)) {
                    rescale_to(mxs);
                    form_p(sc, neg_ref());
                    ps = prob_sum<NT>(pf);
                }
            }
            l_run += ps;
        } else {
            if (__builtin_amdgcn_ballot_w64(mx > m_run + kRescaleSlack)) rescale_to(mx);
        }
        const float neg_m = neg_ref();

        // --- scores of step st+1 (MFMA), then PV of step st (MFMA); bf16
        // forms step st+1's probabilities (VALU) beside the PV MFMAs, fp32
        // forms step st's beside the QK MFMAs.  On the last step the scores
        // (and the probabilities formed from them) come from a stale slot
        // and are discarded.
        if constexpr (sizeof(T) == 2) {
            // An explicit software pipeline over the NF = NQ + NP MFMAs of the
            // step: segment j issues MFMA j, the LDS read of the fragment that
            // MFMA j + kReadLead consumes and, in the PV half, a slice of the
            // next step's probabilities; sched_barrier keeps every segment in
            // place, so each fragment
            // arrives kReadLead MFMAs after its read was issued.  (Left to
            // itself the scheduler, short of registers, reads each fragment
            // right before its MFMA, which then waits out a whole LDS round
            // trip.)  QK MFMAs alternate between the two 32-key tiles and PV
            // MFMAs between the DT output tiles, so consecutive MFMAs never
            // feed each other; every accumulator still sums in the same order.
            // The probabilities of step st+1 are VALU work for the PV
            // segments: group g (pf[g / 2][g % 2], 8 keys of one 32-key tile)
            // is formed from the scores of step st+1 in the DT segments after
            // the last PV MFMA that reads group g of step st, the last group
            // after the loop.  The QK segments carry no VALU work.  The row
            // maxima the reference needs are no longer taken every step (the
            // check at the next step's start, above); against taking them in
            // the PV segments and forming the probabilities beside the QK
            // MFMAs, this is -2.8 % at 128K and -2.7 % at 32K (dense -2.6 %),
            // with bitwise the same output.  The check placed before the
            // step's copies are issued instead was slower than the old way.
            constexpr int NQ = NT * KS, NP = NT * 2 * DT, NF = NQ + NP;
            constexpr int EPP = 8 / DT;   // probabilities per PV segment
            static_assert(EPP * DT == 8 && NP == 2 * NT * DT, "probability groups");
            const T* kb = slot.k((st + 1) & 1);
            const T* vb = slot.v(st & 1);
            auto frag = [&](int j) -> Frag {
                if (j < NQ) return kfrag(kb, j % NT, j / NT);
                const int p = j - NQ;
                return vfrag(vb, p % DT, p / (2 * DT), (p / DT) % 2);
            };
            Frag f[NF];
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) sn[kt] = zero16();
#pragma unroll
            for (int j = 0; j < kReadLead; ++j) f[j] = frag(j);
            __builtin_amdgcn_sched_barrier(0);
            // While a wave issues its MFMA pipeline it takes precedence over
            // the other workgroup's wave on the same SIMD when that one is at
            // its step boundary (copy wait, barrier, copy issue, rescale
            // check), so the matrix pipe is fed first: -0.5 to -0.7 % of the
            // attention time at 32K and 128K against equal priorities.
            __builtin_amdgcn_s_setprio(3);
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                if (j < NQ) {
                    mma(sn[j % NT], f[j], qf[j / NT]);
                } else {
                    const int p = j - NQ;
                    mma(o[p % DT], f[j], pf[p / (2 * DT)][(p / DT) % 2]);
                }
                if (j + kReadLead < NF) f[j + kReadLead] = frag(j + kReadLead);
                if (j >= NQ + DT) {
                    const int p = j - NQ, g = p / DT - 1;
                    if (g < 2 * NT - 1) {
#pragma unroll
                        for (int u = 0; u < EPP; ++u) {
                            const int r = 8 * (g % 2) + EPP * (p % DT) + u;
                            pf[g / 2][g % 2][r & 7] =
                                cvt_p<T>(fast_exp2(fmaf(sn[g / 2][r], sh.scale2, neg_m)));
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_setprio(0);
            // the last group of step st+1's probabilities (with its scores
            // from a stale slot on the last step: formed and discarded)
#pragma unroll
            for (int r = 8; r < 16; ++r)
                pf[NT - 1][1][r & 7] = cvt_p<T>(fast_exp2(fmaf(sn[NT - 1][r], sh.scale2, neg_m)));
        } else {
            // The same MFMA order, six bf16 MFMAs per fragment (see Split3).
            // Segment j issues fragment j's MFMAs beside the split of
            // fragment j + 1 (44 VALU instructions to 192 MFMA cycles) and
            // the LDS read of fragment j + 2.  The QK segments also form this
            // step's probabilities, the PV segments of group g (see above)
            // split those of group g + 1.  Left to the scheduler in one block,
            // the splits ran ahead of the MFMAs: 1057 -> 911 us at 8K (32/8
            // heads, d 128, sparse).
            constexpr int NQ = NT * KS, NP = NT * 2 * DT, NF = NQ + NP;
            constexpr int EPQ = 16 * NT / NQ;   // probabilities per QK segment
            const T* kb = slot.k((st + 1) & 1);
            const T* vb = slot.v(st & 1);
            auto frag = [&](int j) -> Frag {
                if (j < NQ) return kfrag(kb, j % NT, j / NT);
                const int p = j - NQ;
                return vfrag(vb, p % DT, p / (2 * DT), (p / DT) % 2);
            };
#pragma unroll
            for (int kt = 0; kt < NT; ++kt) sn[kt] = zero16();
            float ps[4] = {0.f, 0.f, 0.f, 0.f};
            Op pop[2 * NT];
            Frag f[NF];
            f[0] = frag(0);
            f[1] = frag(1);
            Op cur = key_operand(f[0]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                Op nxt = cur;
                if (j + 2 < NF) f[j + 2] = frag(j + 2);
                if (j + 1 < NF) nxt = key_operand(f[j + 1]);
                if (j < NQ) {
                    mma(sn[j % NT], cur, qf[j / NT]);
#pragma unroll
                    for (int u = 0; u < EPQ; ++u) {
                        const int e = EPQ * j + u, kt = e / 16, r = e % 16;
                        const float pr = fast_exp2(fmaf(sc[kt][r], sh.scale2, neg_m));
                        pf[kt][r >> 3][r & 7] = pr;
                        ps[r & 3] += pr;
                    }
                    if (j == NQ - 1) pop[0] = prob_operand(pf[0][0]);
                } else {
                    const int p = j - NQ, g = p / DT;
                    mma(o[p % DT], cur, pop[g]);
                    if (g + 1 < 2 * NT) {
#pragma unroll
                        for (int u = 0; u < 4 / DT; ++u)
                            split3_pair<true, false>(pop[g + 1], pf[(g + 1) / 2][(g + 1) % 2], p % DT * (4 / DT) + u);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                cur = nxt;
            }
            l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
        }
        // --- mask and max of step st+1 (fp32; bf16 masks at the start of the
        // next step and checks its probabilities there)
        if constexpr (sizeof(T) != 2) {
            if (st + 1 < steps && needs_mask(nb1))
                mask_tail<NT>(sn, qlim - nb1 * B - ((st + 1) % C::NSUB) * C::KT, h);
            mx = tile_max<NT>(sn) * sh.scale2;
        }
        nb0 = nb1;
        nb1 = nb2;
    };
    f32x16 s_alt[NT];
    for (int st = 0; st < steps; st += 2) {
        step(s_cur, s_alt, st);
        if (st + 1 < steps) step(s_alt, s_cur, st + 1);
    }

    float l_tot = halves_sum(l_run);
    if constexpr (G == 2) {
        // the barriers of the longer group's remaining steps, and one more:
        // nobody reads a tile any longer
        for (int st = steps; st <= per * C::NSUB; ++st) __syncthreads();
        const LdsSlots<T> all{slot.k0 - grp * C::K_ELEMS, slot.k1 - grp * C::K_ELEMS,
                              slot.v0 - grp * C::V_ELEMS, slot.v1 - grp * C::V_ELEMS};
        if (grp) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg)
                    *acc_quad<T, D, B>(all, w, dt, rg, lane) = f32x4{
                        o[dt][4 * rg], o[dt][4 * rg + 1], o[dt][4 * rg + 2], o[dt][4 * rg + 3]};
            if (h == 0) ml[32 * w + lc] = steps ? make_float2(m_run, l_tot) : make_float2(kNegInf, 0.f);
        }
        __syncthreads();
        if (grp) return;
        const float2 x = ml[32 * w + lc];
        const float top = fmaxf(m_run, x.x);   // finite: group 0 has an entry, and a row sees a key of it
        const float a = m_run == kNegInf ? 0.f : fast_exp2(m_run - top);
        const float b = x.x == kNegInf ? 0.f : fast_exp2(x.x - top);
        m_run = top;
        l_tot = l_tot * a + x.y * b;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const f32x4 y = *acc_quad<T, D, B>(all, w, dt, rg, lane);
#pragma unroll
                for (int u = 0; u < 4; ++u) o[dt][4 * rg + u] = o[dt][4 * rg + u] * a + y[u] * b;
            }
    }
    const float inv = 1.f / l_tot;
    if constexpr (sizeof(T) == 2 && D == 128 && B == 128) {
        // O through LDS: the wave's 32 x D tile is written to the K slots
        // (free once every wave is done with the last step) and read back as
        // 16-byte row chunks, so that each store writes whole 128-byte lines
        static_assert(2 * 32 * D <= C::K_ELEMS, "two waves' O tiles per K slot");
        if (G == 1) __syncthreads();
        T* ot = (w < 2 ? slot.k(0) : slot.k(1)) + (w & 1) * 32 * D;
        // new to the optimizer: no address of the epilogue is an item-loop
        // invariant kept in a register through the steps
        int ln = lane;
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const float v0 = o[dt][4 * rg + 0] * inv, v1 = o[dt][4 * rg + 1] * inv;
                const float v2 = o[dt][4 * rg + 2] * inv, v3 = o[dt][4 * rg + 3] * inv;
                *reinterpret_cast<uint2*>(ot + line_pos<T, D>(ln & 31, 32 * dt + 8 * rg) + 4 * (ln >> 5)) =
                    make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int r = 4 * it + (ln >> 4), c = (ln & 15) * 8;
            const u32x4 val = *reinterpret_cast<const u32x4*>(ot + line_pos<T, D>(r, c));
            const int tok = m * B + 32 * w + r;
            if (tok < n_tok)
                *reinterpret_cast<u32x4*>(out + (int64_t)tok * sh.o_tok + (int64_t)i * sh.o_head + c) = val;
        }
        if (qvalid && lse && h == 0) lse[(int64_t)i * n_tok + qtok] = (m_run + log2f(l_tot)) * kLn2;
        return;
    }
    if (qvalid) {
        T* orow = out + (int64_t)qtok * sh.o_tok + (int64_t)i * sh.o_head;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
                const int d0 = 32 * dt + 8 * rg + 4 * h;
                const float v0 = o[dt][4 * rg + 0] * inv, v1 = o[dt][4 * rg + 1] * inv;
                const float v2 = o[dt][4 * rg + 2] * inv, v3 = o[dt][4 * rg + 3] * inv;
                if constexpr (sizeof(T) == 2) {
                    *reinterpret_cast<uint2*>(orow + d0) = make_uint2(pack_bf16x2(v0, v1),
                                                                      pack_bf16x2(v2, v3));
                } else {
                    *reinterpret_cast<float4*>(orow + d0) = make_float4(v0, v1, v2, v3);
                }
            }
        }
        if (lse && h == 0) lse[(int64_t)i * n_tok + qtok] = (m_run + log2f(l_tot)) * kLn2;
    }
}

// Persistent kernel: one resident workgroup per slot (2B threads, B/32
// waves); workgroup w starts with item w, then takes the next item of queue
// w % 8 until the queue is empty, then helps drain the other queues.  Taking work dynamically keeps
// every slot busy whatever the mix of list lengths: the hardware dispatcher
// hands workgroups to the shader engines of an XCD in a fixed rotation, so a
// grid of one workgroup per item lets the engines that receive the long items
// hold back all the others.
//
// G = 2, for launches of few items (see attn_d), which last as long as their
// longest list: a workgroup of twice the waves and tiles gives each item's
// list to two groups of waves, half of the entries each, and joins them
// through LDS.  fp32 2K prefill, 8/2 heads, d 64 b 64: 54.9 -> 47.0 us, same box.
template <typename T, int D, int B, bool DENSE, int G>
__global__ __launch_bounds__(2 * B * G, (AttnCfg<T, D, B>::min_waves(G))) void attn_kernel(Shape sh, const T* __restrict__ q,
                                                        const T* __restrict__ kvb,
                                                        const int* __restrict__ block_count,
                                                        const int* __restrict__ block_index,
                                                        T* __restrict__ out,
                                                        float* __restrict__ lse,
                                                        int* __restrict__ queue) {
    typedef AttnCfg<T, D, B> C;
    __shared__ __attribute__((aligned(16))) T ks0[G * C::K_ELEMS];
    __shared__ __attribute__((aligned(16))) T ks1[G * C::K_ELEMS];
    __shared__ __attribute__((aligned(16))) T vs0[G * C::V_ELEMS];
    __shared__ __attribute__((aligned(16))) T vs1[G * C::V_ELEMS];
    __shared__ float2 ml[G == 1 ? 1 : B];
    // the same for every lane of a wave, and known to be: the groups' step
    // counts, and with them their barriers, differ
    const int grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / C::NTH);
    const LdsSlots<T> slot{ks0 + grp * C::K_ELEMS, ks1 + grp * C::K_ELEMS, vs0 + grp * C::V_ELEMS,
                           vs1 + grp * C::V_ELEMS};
    __shared__ int next_item;
    const int per_queue = attn_items(sh) / kNumXcd, own = (int)gridDim.x / kNumXcd;
    // The first item of every workgroup is its own number's (the grid is a
    // multiple of kNumXcd); the counters hand out the rest, so a launch with
    // no more items than workgroups touches none.  Own XCD's queue first; once
    // it is empty, the others with items left in turn (their shortest), so no
    // XCD idles while another still has work.  Whoever finds a queue empty sets
    // its bit in one shared word and learns from it which others are empty
    // too: the last workgroup ends after two round trips, with one request
    // each.  A queue found empty stays empty, and a workgroup tries each once,
    // so the loop ends after at most kNumXcd failures.  K/V copy and attention,
    // sparse, 32/8 heads, against probing every queue / against a load of all
    // counters (eight requests a workgroup, slow with 1024 of them), bf16: d 64
    // b 64 4173 tokens 44.3 / 56.7 -> 42.1 us, d 128 b 64 62.7 / 72.5 -> 59.7, d 128
    // b 128 63.4 / 62.8 -> 60.3; fp32 d 64 b 64 1.5K 47.6 / 45.8 -> 45.0, d 128 b 128
    // 1.5K 96.8 / 92.2 -> 92.3.
    int x = blockIdx.x % kNumXcd, pos = blockIdx.x / kNumXcd, item = x + kNumXcd * pos;
    for (;;) {
        int m, i;
        if (attn_item(sh, item, &m, &i))
            attn_one<T, D, B, DENSE, G>(sh, q, kvb, block_count, block_index, out, lse, m, i, slot, grp, ml);
        if (own == per_queue) break;
        if (threadIdx.x < 64) {   // wave 0
            const int lane = threadIdx.x;
            for (;;) {
                if (lane == 0) pos = own + atomicAdd(queue + x * kQueueStride, 1);
                pos = __builtin_amdgcn_readfirstlane(pos);
                if (pos < per_queue) break;
                int gone = 1 << x;
                if (lane == 0) gone |= atomicOr(queue + kQueueGone, gone);
                const unsigned left = ~__builtin_amdgcn_readfirstlane(gone) & ((1u << kNumXcd) - 1u);
                if (!left) break;
                const unsigned turn = left >> x | left << (kNumXcd - x);
                x = (x + __builtin_ctz(turn)) % kNumXcd;
            }
            if (lane == 0) next_item = pos < per_queue ? x + kNumXcd * pos : -1;
        }
        // the barriers also keep the previous item's LDS reads ahead of the
        // next item's copies
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(next_item);
        __syncthreads();
        if (item < 0) break;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename T, int D, int B>
static hipError_t kvb_t(const Shape& sh, const void* k, const void* v, void* kvb, int* queue,
                        hipStream_t st) {
    hipLaunchKernelGGL((kv_block_kernel<T, D, B>), dim3(sh.mq, sh.hkv), dim3(256), 0, st, sh,
                       (const T*)k, (const T*)v, (T*)kvb, queue);
    return hipGetLastError();
}

hipError_t launch_kv_block(const Shape& sh, const void* k, const void* v, void* kvb, int* queue,
                           hipStream_t st) {
    if (sh.dtype == 0) {
        if (sh.d == 64) return sh.b == 64 ? kvb_t<bf16, 64, 64>(sh, k, v, kvb, queue, st) : kvb_t<bf16, 64, 128>(sh, k, v, kvb, queue, st);
        return sh.b == 64 ? kvb_t<bf16, 128, 64>(sh, k, v, kvb, queue, st) : kvb_t<bf16, 128, 128>(sh, k, v, kvb, queue, st);
    }
    if (sh.d == 64) return sh.b == 64 ? kvb_t<float, 64, 64>(sh, k, v, kvb, queue, st) : kvb_t<float, 64, 128>(sh, k, v, kvb, queue, st);
    return sh.b == 64 ? kvb_t<float, 128, 64>(sh, k, v, kvb, queue, st) : kvb_t<float, 128, 128>(sh, k, v, kvb, queue, st);
}

// Workgroups of `fn` (with `threads` threads) resident on the current device
// at once, rounded down to a multiple of kNumXcd (at least kNumXcd, so that
// every queue has a workgroup).  Cached per (device, kernel).
static int resident_grid(const void* fn, int threads, int* grid) {
    struct Entry { int dev; const void* fn; int grid; };
    static std::mutex mu;
    static std::vector<Entry> cache;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    {
        std::lock_guard<std::mutex> lk(mu);
        for (const Entry& c : cache)
            if (c.dev == dev && c.fn == fn) { *grid = c.grid; return 0; }
    }
    int cus = 0, per_cu = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return (int)e;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, 0);
    if (e != hipSuccess) return (int)e;
    const int g = per_cu * cus / kNumXcd * kNumXcd;
    *grid = g < kNumXcd ? kNumXcd : g;
    std::lock_guard<std::mutex> lk(mu);
    cache.push_back({dev, fn, *grid});
    return 0;
}

constexpr int kSplitItems = 256, kSplitRows = 8;

template <typename T, int D, int B, bool DENSE, int G>
static hipError_t attn_g(const Shape& s, const dim3& grid, const void* q, const void* kvb,
                         const int* bc, const int* bi, void* out, float* lse, int* queue,
                         hipStream_t st) {
    hipLaunchKernelGGL((attn_kernel<T, D, B, DENSE, G>), grid, dim3(2 * B * G), 0, st, s,
                       (const T*)q, (const T*)kvb, bc, bi, (T*)out, lse, queue);
    return hipGetLastError();
}

template <typename T, int D, int B, bool DENSE>
static hipError_t attn_d(const Shape& s, const void* q, const void* kvb, const int* bc,
                         const int* bi, void* out, float* lse, int* queue, hipStream_t st) {
    int g = 0;
    // Lists are split while there are no more items than the MI355X has CUs,
    // and at least kSplitRows block rows.  K/V copy and attention, sparse and
    // dense, whole -> split: 256 items, 8 heads of 32 block rows, fp32 d 64
    // b 64 51.4 -> 34.6 and 101.5 -> 62.2 us, fp32 d 128 b 64 89.7 -> 58.2 and
    // 183 -> 110 us, bf16 d 128 b 64 27.4 -> 23.2 and 48.1 -> 35.0 us; 32 heads
    // of 8 block rows, fp32 d 64 b 64 22.9 -> 19.5 and 40.7 -> 31.3 us, bf16 d 128
    // b 64 17.5 -> 16.8 and 30.1 -> 25.3 us.  Up to 4 block rows the join takes
    // what the shorter chain gives (bf16 d 128 b 64 dense 18.9 -> 21.3 us), and
    // so it does with lists of a few blocks on either side of the line (one
    // head of 100 rows, fp32 d 128 b 64 18.4 -> 21.0 us, bf16 10.3 -> 12.0; at
    // worst 28 heads of 9 rows, bf16 d 64 b 128, 16.6 -> 21.0 us), which the host
    // cannot see.  Past 256 items, 257 to 512 of them, dense calls would gain
    // up to 45 % (28 and 32 heads at b 128: -33 to +9 %), sparse ones lose as
    // often as they gain: bf16 d 64 b 64 -24 to +18 %, d 128 b 64 -27 to +11 %,
    // d 64 b 128 +9 to +61 %; fp32 d 64 b 64 -30 to +23 %, d 128 b 64 -36 to
    // +41 %, d 64 b 128 -23 to +41 %.  The items counted are the (head, row) pairs,
    // so that no work order changes a result, and dense and sparse follow one
    // rule.
    if constexpr (AttnCfg<T, D, B>::CAN_SPLIT) {
        if (s.mq >= kSplitRows && (int64_t)s.hq * s.mq <= kSplitItems) {
            const int e = resident_grid((const void*)attn_kernel<T, D, B, DENSE, 2>, 4 * B, &g);
            if (e) return (hipError_t)e;
            return attn_g<T, D, B, DENSE, 2>(s, dim3((unsigned)std::min(g, attn_items(s))), q, kvb, bc,
                                             bi, out, lse, queue, st);
        }
    }
    const int e = resident_grid((const void*)attn_kernel<T, D, B, DENSE, 1>, 2 * B, &g);
    if (e) return (hipError_t)e;
    return attn_g<T, D, B, DENSE, 1>(s, dim3((unsigned)std::min(g, attn_items(s))), q, kvb, bc, bi,
                                     out, lse, queue, st);
}

template <typename T, int D, int B>
static hipError_t attn_t(const Shape& sh, bool dense, const void* q, const void* kvb,
                         const int* bc, const int* bi, void* out, float* lse, int* queue,
                         hipStream_t st) {
    if (!dense) return attn_d<T, D, B, false>(sh, q, kvb, bc, bi, out, lse, queue, st);
    Shape s = sh;
    s.attn_order = sh.attn_order_dense;
    return attn_d<T, D, B, true>(s, q, kvb, bc, bi, out, lse, queue, st);
}

hipError_t launch_attention(const Shape& sh, bool dense, const void* q, const void* kvb,
                            const int* bc, const int* bi, void* out, float* lse, int* queue,
                            hipStream_t st) {
    if (sh.dtype == 0) {
        if (sh.d == 64) return sh.b == 64 ? attn_t<bf16, 64, 64>(sh, dense, q, kvb, bc, bi, out, lse, queue, st)
                                          : attn_t<bf16, 64, 128>(sh, dense, q, kvb, bc, bi, out, lse, queue, st);
        return sh.b == 64 ? attn_t<bf16, 128, 64>(sh, dense, q, kvb, bc, bi, out, lse, queue, st)
                          : attn_t<bf16, 128, 128>(sh, dense, q, kvb, bc, bi, out, lse, queue, st);
    }
    if (sh.d == 64) return sh.b == 64 ? attn_t<float, 64, 64>(sh, dense, q, kvb, bc, bi, out, lse, queue, st)
                                      : attn_t<float, 64, 128>(sh, dense, q, kvb, bc, bi, out, lse, queue, st);
    return sh.b == 64 ? attn_t<float, 128, 64>(sh, dense, q, kvb, bc, bi, out, lse, queue, st)
                      : attn_t<float, 128, 128>(sh, dense, q, kvb, bc, bi, out, lse, queue, st);
}

}  // namespace pa
