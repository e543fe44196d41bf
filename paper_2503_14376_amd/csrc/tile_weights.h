// The weighted intra-chunk matrix of a tiled kernel (bf16) in memory, for contractions that are too wide for a wavefront
// to hold its rows of X in registers:
//   E[r][c] = exp2(wrow[r] + wcol[c]) * (X_r . Y_c)     within a chunk, c <= r (dV: c >= r), rounded to bf16,
// as (BH, Nc, L, L), and for H of mLSTMexp the sums of its rows in fp32, one per row and block of columns.  The tiled kernels
// then read it (NOE == 2 in tile_fast.h) where they would form it.
// A workgroup forms one block of 32 NW x 32 NW values; both operands arrive in slices of 64 contraction columns through a ring of
// asynchronous loads, as in tile_fast.h.  Blocks beyond the diagonal are not launched.
// Bound by how fast the slices arrive: 16 heads of 1024, 4096 steps, chunk 256 65 - 79 us per launch (H, whose row sums come on top,
// the longest), 403 MB of slices (268 MB of operands once) and 25 MB of E, 5.4 - 6.6 TB/s together.
#pragma once
#include "lds_tiles.h"
#include "tfla_internal.h"

namespace tfla {

// PAD: as in tile_fast.h.
template <int NW, int MODE, int PAD>
__global__ void __launch_bounds__(NW * 64) weights_kernel_bf16(TileArgs a) {
    using E = Elem<bf16_t>;
    using frag = E::frag;
    constexpr bool UPPER = (MODE & 1) != 0;
    constexpr int NT = NW * 64, BR = NW * 32, NB = NW, BS = 64, KSS = BS / 16, NS = 4;
    constexpr int XB = BR * BS * 2, STAGE = 2 * XB;
    __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];
    using DT = DmaTile<BR, BS, NT, SWZ_K>;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
    const int gy = a.L / BR;
    unsigned rem;
    unsigned wg = tile_divmod(xcd_remap(blockIdx.x, gridDim.x), (unsigned)(gy * (gy + 1) / 2), -1, rem);
    // block pair number rem of the triangle: (far, near) with near <= far
    int far = 0, near = __builtin_amdgcn_readfirstlane((int)rem);
    while (near > far) { ++far; near -= far; }
    const int rb = UPPER ? near : far, cb = UPPER ? far : near;
    const unsigned bhn = (unsigned)a.dec_bh, bpx = (unsigned)a.dec_bpx;
    wg = tile_divmod(wg, bpx, a.sh_bpx, rem);
    const unsigned bl = rem;
    wg = tile_divmod(wg, (unsigned)a.Nc, a.sh_nc, rem);
    const int kc = __builtin_amdgcn_readfirstlane((int)rem);
    const int bh = __builtin_amdgcn_readfirstlane((int)(wg * bpx + bl));
    const long tbase = (long)bh * a.T + (long)kc * a.L;
    const int r0 = rb * BR, c0 = cb * BR, wr0 = r0 + wave * 32;
    const int xld = PAD ? a.in_ld1 : a.d1;
    const long tin = PAD ? (long)bh * a.out_T + (long)kc * a.L : tbase;
    const int steps_left = PAD ? a.out_T - kc * a.L : 0;       // of the sequence, from the first step of the chunk on
    const bf16_t* X = reinterpret_cast<const bf16_t*>(a.X) + (tin + r0) * xld;
    const bf16_t* Y = reinterpret_cast<const bf16_t*>(a.Y) + (tin + c0) * xld;
    const int NI = a.d1 / BS;
    const uint32_t smem_a = lds_addr(smem);

    // the weights' exponents: older than the ring's requests, so that the wait for them, after the products, is none
    const float wr = a.wrow[tbase + wr0 + l32];
    f32x4 wc[NB][4];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int q = 0; q < 4; ++q) wc[nb][q] = *reinterpret_cast<const f32x4*>(a.wcol + tbase + c0 + 32 * nb + 8 * q + 4 * g);

    DT dt;  dt.init(xld, tid);
    auto issue = [&](int i, uint32_t st) {
        if constexpr (PAD) {
            const int cl = a.in_ld1 - i * BS;
            dt.template issue_bounded<true>(X + i * BS, bounded_bytes(steps_left - r0, cl, 2 * xld), cl, st, tid);
            dt.template issue_bounded<true>(Y + i * BS, bounded_bytes(steps_left - c0, cl, 2 * xld), cl, st + XB, tid);
        } else {
            dt.issue(X + i * BS, st, tid);
            dt.issue(Y + i * BS, st + XB, tid);
        }
    };
    for (int p = 0; p < NS - 1 && p < NI; ++p) issue(p, smem_a + p * STAGE);

    f32x16 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nb][v] = 0.0f;
    KFragReader<BS> rd;  rd.init(l32, g);
    int slot = 0;
    for (int i = 0; i < NI; ++i) {
        if (i + NS - 2 < NI) wait_vmcnt<(NS - 2) * 2 * DT::N>();
        else wait_vmcnt_dyn((NI - 1 - i) * 2 * DT::N);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (the fragment reads of the slice before have left its stage)
        barrier_nofence();
        const char* sb = smem + slot * STAGE;
        // slice i + NS - 1 goes into the stage of slice i - 1
        if (i + NS - 1 < NI) issue(i + NS - 1, smem_a + (uint32_t)(slot == 0 ? NS - 1 : slot - 1) * STAGE);
        if (++slot == NS) slot = 0;
#pragma unroll
        for (int ks = 0; ks < KSS; ++ks) {
            frag x, y[NB];
            x.v = rd.load(sb, ks, wave);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) y[nb].v = rd.load(sb + XB, ks, nb);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb] = E::mma(y[nb], x, acc[nb]);
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_nofence();                                   // every wave is done reading the ring

    // as in tile_fast.h: lane = row l32 of the wavefront's, register v of block nb = column 32 nb + acc_row(v, g)
    constexpr int OCPR = BR / 8, ORB = BR * 2;
    char* otile = smem + wave * (32 * ORB);
    const int fsw = swz_mask<SWZ_K, OCPR>(l32);
    const bool diag = rb == cb;
    float rowsum = 0.0f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        float p[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            p[v] = acc[nb][v] * fast_exp2(wr + wc[nb][v >> 2][v & 3]);
            const int c = 32 * nb + acc_row(v, g), r = 32 * wave + l32;
            if (diag && (UPPER ? c < r : c > r)) p[v] = 0.0f;
            if (MODE == MODE_H) rowsum += p[v];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *reinterpret_cast<uint2*>(otile + l32 * ORB + (((4 * nb + j) ^ fsw) * 16) + 8 * g) =
                uint2{pack_bf16x2(p[4 * j], p[4 * j + 1]), pack_bf16x2(p[4 * j + 2], p[4 * j + 3])};
    }
    if (MODE == MODE_H) {
        if (a.variant == 0) {
            rowsum += __shfl_xor(rowsum, 32, 64);
            if (g == 0) a.nrm_out[(long)cb * (long)bhn * a.T + tbase + wr0 + l32] = rowsum;
        }
    }
    constexpr int RPI = 64 / OCPR;
    char* ebase = reinterpret_cast<char*>(a.E) + ((((long)bh * a.Nc + kc) * a.L + wr0) * a.L + c0) * 2;
#pragma unroll
    for (int q = 0; q < 32 / RPI; ++q) {
        const int r = q * RPI + lane / OCPR, c = lane % OCPR;
        const u32x4 w = *reinterpret_cast<const u32x4*>(otile + r * ORB + ((c ^ swz_mask<SWZ_K, OCPR>(r)) * 16));
        *reinterpret_cast<u32x4*>(ebase + (long)r * a.L * 2 + c * 16) = w;
    }
}

}  // namespace tfla
