// Device-side building blocks shared by the ProxyAttn kernels (gfx950).
//
// Matrix products use the 32x32 MFMA tile.  For a product D = A * B with
// A: 32 x 16 and B: 16 x 32, lane l (64 lanes) supplies
//     A[m = l % 32][k-slot (l / 32, j)]   and   B[k-slot (l / 32, j)][n = l % 32]
// for j = 0..7, and receives D[m][n = l % 32] for the 16 rows
//     m = 8 * (r / 4) + 4 * (l / 32) + (r % 4),  r = 0..15.
// Which hardware k index a (half, j) slot maps to does not matter as long as
// both operands use the same slot for the same k; every kernel here fills A
// and B through that one slot convention.
//
// bf16 operands: one v_mfma_f32_32x32x16_bf16 per 16-wide k step.
// fp32 operands: each is split into three bf16 terms, and six such MFMAs per
// step form the product (see Split3); the data layout of every kernel is
// identical for the two element types.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pa {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// 16 bytes as a native vector: register staging of tiles (HIP's uint4 class
// defeats scalar replacement and ends up on the stack)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Element e of a 16-byte vector holding 16/sizeof(T) values of T.
template <typename T> __device__ __forceinline__ void put_elem(u32x4& x, int e, T v);
template <> __device__ __forceinline__ void put_elem<float>(u32x4& x, int e, float v) {
    x[e] = __float_as_uint(v);
}
template <> __device__ __forceinline__ void put_elem<__bf16>(u32x4& x, int e, __bf16 v) {
    const uint32_t b = __builtin_bit_cast(uint16_t, v);
    x[e >> 1] |= (e & 1) ? (b << 16) : b;
}

// Element e of such a vector as a float.
template <typename T> __device__ __forceinline__ float get_elem(const u32x4& x, int e);
template <> __device__ __forceinline__ float get_elem<float>(const u32x4& x, int e) {
    return __uint_as_float(x[e]);
}
template <> __device__ __forceinline__ float get_elem<__bf16>(const u32x4& x, int e) {
    const uint32_t w = x[e >> 1];
    return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
}

__device__ __forceinline__ u32x4 zero_u32x4() {
    u32x4 z = {0u, 0u, 0u, 0u};
    return z;
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kNegInf = -__builtin_huge_valf();

template <typename T> struct FragOf;
template <> struct FragOf<bf16> { typedef bf16x8 type; };
template <> struct FragOf<float> { typedef f32x8 type; };

// Elements of T per 16-byte vector load.
template <typename T> struct Vec16 { static constexpr int n = 16 / sizeof(T); };

__device__ __forceinline__ void mma(f32x16& acc, const bf16x8& a, const bf16x8& b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}

// fp32 operands as three bf16 terms, x = hi + mid + lo: hi the top 8 significant
// bits, by truncation (no finite x overflows, and one permute makes two) or, with
// NEAR, to nearest; mid and lo by rounding what is left.  The sum is exact for
// |x| >= 2^-110; below, bits under bf16's smallest denormal go, 2^-134 at most.
// |mid| <= 2^-7 and |lo| <= 2^-16 of x's power of two with hi truncated, half of
// each with hi to nearest, so the three products of nine that are left out stay
// below 2^-23 of x y where one operand's hi is to nearest (2^-22 where neither
// is): queries and probabilities are rounded, keys and values, which the inner
// loops split, truncated.  Rounding those too takes two
// more clamps a pair and 6-8 % more time (8K sparse, d 128: 927 -> 993 us), the
// two next products in their place 12-16 %, for errors against 64 bits that are
// the same on the timed cases.
// Six bf16 MFMAs of 16 k each take 192 cycles where eight fp32 MFMAs of 2 k took
// 512, and round the accumulator six times instead of eight, but by truncation.
// Errors against 64 bits, fp32 MFMAs -> split: attention outputs 1.08e-6 ->
// 8.5e-7 (3K, d 128) and 8.8e-7 -> 6.4e-7 (2K, d 64), block scores 1.08e-7 ->
// 9.5e-8 (4K), means of 24 inputs; a dot product of 64 normal deviates, in units
// of 2^-24 of its absolute sum, largest 2.5 -> 2.3, rms 0.47 -> 0.37; a single
// product, largest 1.6 -> 2.8 (6.3 with both operands truncated), rms 0.60 -> 0.72.
// Sparse attention 8K, 32/8 heads, d 128: 1340 -> 911 us, dense d 64 b 64 5K: 543
// -> 347 us, estimate 8K: 128 -> 96 us.
struct Split3 {
    bf16x8 hi, mid, lo;
};
// Elements 2 j and 2 j + 1.  CLAMP keeps a value that would round past the
// largest bf16 at it.
template <bool NEAR, bool CLAMP>
__device__ __forceinline__ void split3_pair(Split3& s, const f32x8& x, int j) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const float xa = x[2 * j], xb = x[2 * j + 1];
    const uint32_t a = __float_as_uint(xa), b = __float_as_uint(xb);
    bf16x2 hi;
    uint32_t ha, hb;
    if constexpr (NEAR) {
        const float top = CLAMP ? __uint_as_float(0x7f7f0000u) : 0.f;
        const f32x2 c = {CLAMP ? __builtin_amdgcn_fmed3f(xa, -top, top) : xa,
                         CLAMP ? __builtin_amdgcn_fmed3f(xb, -top, top) : xb};
        hi = __builtin_convertvector(c, bf16x2);
        const uint32_t h = __builtin_bit_cast(uint32_t, hi);
        ha = h << 16;
        hb = h & 0xffff0000u;
    } else {
        hi = __builtin_bit_cast(bf16x2, __builtin_amdgcn_perm(b, a, 0x07060302u));
        ha = a & 0xffff0000u;
        hb = b & 0xffff0000u;
    }
    const f32x2 r = {xa - __uint_as_float(ha), xb - __uint_as_float(hb)};
    const bf16x2 mid = __builtin_convertvector(r, bf16x2);
    const uint32_t m = __builtin_bit_cast(uint32_t, mid);
    const f32x2 t = {r[0] - __uint_as_float(m << 16), r[1] - __uint_as_float(m & 0xffff0000u)};
    const bf16x2 lo = __builtin_convertvector(t, bf16x2);
    s.hi[2 * j] = hi[0];
    s.hi[2 * j + 1] = hi[1];
    s.mid[2 * j] = mid[0];
    s.mid[2 * j + 1] = mid[1];
    s.lo[2 * j] = lo[0];
    s.lo[2 * j + 1] = lo[1];
}
template <bool NEAR, bool CLAMP>
__device__ __forceinline__ Split3 split3(const f32x8& x) {
    Split3 s;
#pragma unroll
    for (int j = 0; j < 4; ++j) split3_pair<NEAR, CLAMP>(s, x, j);
    return s;
}
// The six products, smallest first.
__device__ __forceinline__ void mma(f32x16& acc, const Split3& a, const Split3& b) {
    mma(acc, a.lo, b.hi);
    mma(acc, a.hi, b.lo);
    mma(acc, a.mid, b.mid);
    mma(acc, a.mid, b.hi);
    mma(acc, a.hi, b.mid);
    mma(acc, a.hi, b.hi);
}

// Fragments as the MFMAs take them: bf16 as they are, fp32 split.  One operand
// of every product is a key or value, the other a query or a probability
// (at most 2^8: nothing to clamp).
template <typename T> struct OperandOf { typedef bf16x8 type; };
template <> struct OperandOf<float> { typedef Split3 type; };
__device__ __forceinline__ bf16x8 key_operand(const bf16x8& f) { return f; }
__device__ __forceinline__ Split3 key_operand(const f32x8& f) { return split3<false, false>(f); }
__device__ __forceinline__ bf16x8 query_operand(const bf16x8& f) { return f; }
__device__ __forceinline__ Split3 query_operand(const f32x8& f) { return split3<true, true>(f); }
__device__ __forceinline__ Split3 prob_operand(const f32x8& f) { return split3<true, false>(f); }

template <typename T>
__device__ __forceinline__ typename FragOf<T>::type load_frag(const T* p) {
    return *reinterpret_cast<const typename FragOf<T>::type*>(p);
}

// LDS tiles that MFMA fragments are read from: lines of D elements whose
// 16-byte chunks are XOR-ed in position so that the 16 lanes an LDS read
// serves at a time, which take one chunk index of 16 consecutive lines, meet
// all 16 bank groups (256 bytes): lines of 16 or more chunks by line % 16,
// lines of 8 chunks (two to a bank sweep) by line / 2 % 8.  No bank conflicts,
// as with lines padded by a chunk each, but no padding to copy or to hold, and
// a tile is one contiguous run for global -> LDS copies.
template <int P>
__device__ __forceinline__ int chunk_xor(int line) {
    static_assert(P >= 8, "lines of at least 8 chunks");
    return P >= 16 ? line & 15 : line / 2 & 7;
}
template <typename T, int D>
__device__ __forceinline__ int line_pos(int line, int elem) {
    constexpr int V = Vec16<T>::n;
    return line * D + ((elem / V) ^ chunk_xor<D / V>(line)) * V;
}

// A lane's fragment reads from tile lines (see line_pos): 8 consecutive
// elements, one chunk of bf16 or two of fp32, of line lc (+ 32, + 64, ...).
// The XOR touches at most the low four bits of the chunk number, so NX
// offsets serve every fragment of both tiles; the rest is an immediate.
template <typename T, int D>
struct LaneLines {
    static constexpr int V = Vec16<T>::n;
    static constexpr int SPAN = D / V >= 16 ? 16 : 8;   // chunks that the XOR mixes
    static constexpr int NX = SPAN / 2;
    int x[NX];   // byte offsets: bf16 chunk 2 u + h, fp32 chunk 4 (u / 2) + 2 h + u % 2
    __device__ __forceinline__ LaneLines(int lc, int h) {
#pragma unroll
        for (int u = 0; u < NX; ++u)
            x[u] = line_pos<T, D>(lc, (V == 8 ? 2 * u + h : 4 * (u / 2) + 2 * h + u % 2) * V) *
                   (int)sizeof(T);
    }
    // Makes the offsets new to the optimizer.  Called in every step: it would
    // otherwise keep offset + tile address, loop invariants, in registers for
    // each of the four tiles, where the read's immediate holds the tile's.
    __device__ __forceinline__ void renew() {
#pragma unroll
        for (int u = 0; u < NX; ++u) asm volatile("" : "+v"(x[u]));
    }
    // elements f + 8 h .. + 7 of the line, f a multiple of 16
    __device__ __forceinline__ typename FragOf<T>::type frag(const T* tile, int f) const {
        constexpr int SE = SPAN * V;   // elements the XOR mixes
        const char* t = reinterpret_cast<const char*>(tile + f / SE * SE);
        const int u = f % SE / 16;
        if constexpr (V == 8) {
            return *reinterpret_cast<const typename FragOf<T>::type*>(t + x[u]);
        } else {
            const f32x4 a = *reinterpret_cast<const f32x4*>(t + x[2 * u]);
            const f32x4 b = *reinterpret_cast<const f32x4*>(t + x[2 * u + 1]);
            return f32x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        }
    }
};

// Waits for this wave's global -> LDS copies (they count in vmcnt, like any
// vector-memory load).  A copy's data is in LDS only once its wave has
// waited; the barrier after this wait then hands the tiles to the other
// waves.  (s_waitcnt fields: vmcnt 0, expcnt and lgkmcnt left at their
// maxima.)
__device__ __forceinline__ void wait_copies() { __builtin_amdgcn_s_waitcnt(0x0F70); }

__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}

// Row (within a 32-row C tile) held in accumulator slot r by lane half h.
__device__ __forceinline__ int c_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// Round-to-nearest-even fp32 -> bf16 (finite inputs).
__device__ __forceinline__ bf16 f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    uint16_t h = (uint16_t)(u >> 16);
    return __builtin_bit_cast(bf16, h);
}

// Two fp32 values rounded to bf16 (nearest-even) packed low-first in 32 bits.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return (uint32_t)__builtin_bit_cast(uint16_t, f32_to_bf16_rne(lo)) |
           ((uint32_t)__builtin_bit_cast(uint16_t, f32_to_bf16_rne(hi)) << 16);
}

__device__ __forceinline__ float bf16_to_f32(bf16 x) {
    uint16_t h = __builtin_bit_cast(uint16_t, x);
    return __uint_as_float(((uint32_t)h) << 16);
}

template <typename T> __device__ __forceinline__ float to_f32(T x);
template <> __device__ __forceinline__ float to_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f32<bf16>(bf16 x) { return bf16_to_f32(x); }

template <typename T> __device__ __forceinline__ T from_f32_rne(float x);
template <> __device__ __forceinline__ float from_f32_rne<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16 from_f32_rne<bf16>(float x) { return f32_to_bf16_rne(x); }

// 2^x on the hardware transcendental unit (v_exp_f32, ~1 ulp; no denormal
// range fix-up, which the softmax does not need).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Exchanges between the two wave halves without LDS: v_permlane32_swap of x
// with itself gives, in every lane l, r[0] = x[l % 32] and r[1] = x[l % 32 + 32].
__device__ __forceinline__ float swap_halves(float x) {   // x of lane l ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    return __uint_as_float((__lane_id() & 32) ? r[0] : r[1]);
}
__device__ __forceinline__ float halves_max(float x) {    // max of lanes l and l ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float halves_sum(float x) {    // x[l % 32] + x[l % 32 + 32]
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// Monotone map of a float to uint32 (larger float -> larger key).
__device__ __forceinline__ uint32_t float_order_key(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Index of the lower-triangular pair (m, n), n <= m.
__device__ __forceinline__ int64_t tri_index(int m, int n) {
    return (int64_t)m * (m + 1) / 2 + n;
}

}  // namespace pa
