// Device-side building blocks for the gfx950 mLSTM kernels: MFMA fragments, LDS staging
// (natural and transposed), small wavefront reductions.
//
// Fragment convention used by every kernel here.  A "fragment" is 8 consecutive elements
// along the contraction index k that one lane feeds to the matrix core: lane l (0..63) of a
// 32x32 MFMA owns row/column (l & 31) of its operand and the k-group (l >> 5).  For bf16
// one fragment is the 8xbf16 operand of v_mfma_f32_32x32x16_bf16 (k = 16*step + 8*group + e);
// for fp32 the same 8 elements are fed one at a time to eight v_mfma_f32_32x32x2_f32.
// Both operands of a product use the same (step, group, e) -> k mapping, so the result does
// not depend on which k each slot really is.  The 32x32 fp32 result keeps, in register v of
// lane l, element (row 8*(v/4) + 4*(l>>5) + (v&3), column l & 31).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tfla {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int acc_row(int v, int grp) { return 8 * (v >> 2) + 4 * grp + (v & 3); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// sigma(x) of a bf16 value, as close as the library's exponential and an IEEE division come (over all 65536 values at most
// 1.59 ulp of fp32 and 0.064 on average, both ways), in 17 vector instructions instead of 28.
// e = exp(-|x|) = 2^n 2^f with f in [-1/2, 1/2] from a two-term product with log2 e; below -128, where e is zero, the
// argument stays finite.  The denominator lies in [1, 2], so the division needs none of the scaling and special cases of the
// general one: the quotient by the hardware's reciprocal, and its remainder once more.
// (The hardware's exp2 of -x log2 e and its reciprocal alone are three instructions, but their relative error grows with
// |x|, to 5e-6 at x = -80, and nothing is left below -88.)
__device__ __forceinline__ float sigmoid_bf16(float x) {
    float a = -fabsf(x);
    a = a < -128.0f ? -128.0f : a;
    const float n = rintf(a * 1.44269502e+00f);
    const float f = __builtin_fmaf(a, 1.92596299e-08f, __builtin_fmaf(a, 1.44269502e+00f, -n));
    const float e = __builtin_amdgcn_ldexpf(fast_exp2(f), (int)n);
    const float d = 1.0f + e, m = x >= 0.0f ? 1.0f : e, r = __builtin_amdgcn_rcpf(d), q = m * r;
    return __builtin_fmaf(__builtin_fmaf(-d, q, m), r, q);
}

__device__ __forceinline__ uint32_t bf16_bits_rne(float x) {
    // round-to-nearest-even conversion, as bits in the low half
    bf16_t b = (bf16_t)x;
    return (uint32_t)__builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float bf16_lo_to_f32(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi_to_f32(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// two fp32 values -> one dword of two bf16 (round to nearest even), a single v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    bf16x2 v = {(bf16_t)lo, (bf16_t)hi};
    return __builtin_bit_cast(uint32_t, v);
}

template <typename DT> struct Elem;

template <> struct Elem<bf16_t> {
    static constexpr int PAD = 8;  // elements of padding per LDS row (16 bytes)
    struct frag { bf16x8 v; };
    static __device__ __forceinline__ frag load(const bf16_t* p) {
        frag f; f.v = *reinterpret_cast<const bf16x8*>(p); return f;
    }
    static __device__ __forceinline__ f32x16 mma(const frag& a, const frag& b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
    }
    static __device__ __forceinline__ frag pack(const float* p) {
        frag f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f.v[e] = (bf16_t)p[e];
        return f;
    }
    static __device__ __forceinline__ float to_f32(bf16_t x) { return (float)x; }
    static __device__ __forceinline__ bf16_t from_f32(float x) { return (bf16_t)x; }
    static __device__ __forceinline__ float frag_elem(const frag& f, int e) { return (float)f.v[e]; }
};

template <> struct Elem<float> {
    static constexpr int PAD = 4;
    struct frag { float v[8]; };
    static __device__ __forceinline__ frag load(const float* p) {
        frag f;
        f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { f.v[e] = a[e]; f.v[4 + e] = b[e]; }
        return f;
    }
    static __device__ __forceinline__ frag zero() {
        frag f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f.v[e] = 0.0f;
        return f;
    }
    static __device__ __forceinline__ f32x16 mma(const frag& a, const frag& b, f32x16 c) {
#pragma unroll
        for (int e = 0; e < 8; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[e], b.v[e], c, 0, 0, 0);
        return c;
    }
    static __device__ __forceinline__ frag pack(const float* p) {
        frag f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f.v[e] = p[e];
        return f;
    }
    static __device__ __forceinline__ float to_f32(float x) { return x; }
    static __device__ __forceinline__ float from_f32(float x) { return x; }
    static __device__ __forceinline__ float frag_elem(const frag& f, int e) { return f.v[e]; }
};

// Source row of slot (8*u + e) of a transposed tile.  With PERM the eight rows of a group
// are those that registers 8c..8c+7 of a 32x32 MFMA result hold for lane group g, so that a
// result tile can be fed back as an operand against this tile without leaving registers.
template <bool PERM> __device__ __forceinline__ int tr_src_row(int u, int e) {
    if (!PERM) return 8 * u + e;
    const int st = u >> 2, c = (u >> 1) & 1, g = u & 1;
    return 32 * st + 16 * c + 4 * g + (e & 3) + 8 * (e >> 2);
}

// ---------------------------------------------------------------------------------------
// Staging of the fp32 kernels' tiles, in their own row-major layout or transposed (contraction index contiguous per
// LDS row): load() issues the global loads into registers, store() writes them to LDS later, so the loads of the next tile are in flight
// while the current tile is being multiplied.
// ---------------------------------------------------------------------------------------
template <typename DT, int ROWS, int COLS, int NT> struct RowsPrefetch {
    static constexpr int EPC = 16 / (int)sizeof(DT), CPR = COLS / EPC, TOTAL = ROWS * CPR;
    static constexpr int N = (TOTAL + NT - 1) / NT;
    u32x4 r[N];
    // PAD: only rows_left rows and cols_left columns exist from the tile's first on, the rest reads as zero
    template <bool PAD = false>
    __device__ __forceinline__ void load(const DT* g, long gstride, int tid, int rows_left = 0, int cols_left = 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * NT;
            if (TOTAL % NT == 0 || c < TOTAL) {
                if (PAD && (c / CPR >= rows_left || (c % CPR) * EPC >= cols_left)) r[i] = u32x4{0u, 0u, 0u, 0u};
                else r[i] = *reinterpret_cast<const u32x4*>(g + (long)(c / CPR) * gstride + (c % CPR) * EPC);
            }
        }
    }
    __device__ __forceinline__ void store(DT* lds, int lstride, int tid) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int c = tid + i * NT;
            if (TOTAL % NT == 0 || c < TOTAL)
                *reinterpret_cast<u32x4*>(lds + (c / CPR) * lstride + (c % CPR) * EPC) = r[i];
        }
    }
};

template <typename DT, int ROWS, int COLS, int NT, bool PERM> struct TrPrefetch;

template <int ROWS, int COLS, int NT, bool PERM> struct TrPrefetch<float, ROWS, COLS, NT, PERM> {
    static constexpr int UNITS = (ROWS / 8) * COLS, N = (UNITS + NT - 1) / NT;
    float w[N][8];
    template <bool PAD = false>
    __device__ __forceinline__ void load(const float* g, long gstride, int tid, int rows_left = 0, int cols_left = 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int idx = tid + i * NT;
            if (UNITS % NT == 0 || idx < UNITS) {
                const int col = idx % COLS, u = idx / COLS;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int row = tr_src_row<PERM>(u, e);
                    w[i][e] = (PAD && (row >= rows_left || col >= cols_left)) ? 0.0f : g[(long)row * gstride + col];
                }
            }
        }
    }
    __device__ __forceinline__ void store(float* lds, int lstride, int tid) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int idx = tid + i * NT;
            if (UNITS % NT == 0 || idx < UNITS) {
                const int col = idx % COLS, u = idx / COLS;
                f32x4 a = {w[i][0], w[i][1], w[i][2], w[i][3]}, b = {w[i][4], w[i][5], w[i][6], w[i][7]};
                *reinterpret_cast<f32x4*>(lds + col * lstride + 8 * u) = a;
                *reinterpret_cast<f32x4*>(lds + col * lstride + 8 * u + 4) = b;
            }
        }
    }
};

// four consecutive values as one store
__device__ __forceinline__ void store4(float* p, float a, float b, float c, float d) {
    f32x4 w = {a, b, c, d};
    *reinterpret_cast<f32x4*>(p) = w;
}

// Workgroups are handed to the 8 XCDs round-robin by their linear id.  This remaps the
// hardware id so that each XCD (and its L2) works on a contiguous range of logical ids.
__device__ __forceinline__ unsigned xcd_remap(unsigned hw, unsigned total) {
    if (total % 8u != 0u) return hw;
    return (hw % 8u) * (total / 8u) + hw / 8u;
}

// ---------------------------------------------------------------------------------------
// Wavefront helpers (64 lanes)
// ---------------------------------------------------------------------------------------
// Sum over groups of N neighbouring lanes (N = 2 ... 64, aligned), in every lane, without going through LDS (a shuffle by
// ds_bpermute is a round trip of some hundred clocks): lanes 1 and 2 apart by quad permutations, the other half of a
// group of 8 and of 16 by mirroring it (its lanes all hold the same sum by then), rows of 16 and halves of 32 by the
// swap instructions, which given the same value twice return the two sides of each pair.
template <int CTRL> __device__ __forceinline__ float dpp_move(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int N> __device__ __forceinline__ float lanes_sum(float x) {
    if constexpr (N >= 2) x += dpp_move<0xb1>(x);       // quad_perm [1, 0, 3, 2]
    if constexpr (N >= 4) x += dpp_move<0x4e>(x);       // quad_perm [2, 3, 0, 1]
    if constexpr (N >= 8) x += dpp_move<0x141>(x);      // row_half_mirror
    if constexpr (N >= 16) x += dpp_move<0x140>(x);     // row_mirror
    if constexpr (N >= 32) {
        const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
        const unsigned lo = p[0], hi = p[1];
        x = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
    }
    if constexpr (N >= 64) {
        const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
        const unsigned lo = p[0], hi = p[1];
        x = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
    }
    return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
    return x;
}
// sum over the 32 lanes that share (lane >> 5)
__device__ __forceinline__ float half_sum(float x) {
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

}  // namespace tfla
