// fp32 path of the intra-chunk tiled kernels (see tile.hip for what is computed): operands staged through registers.
#pragma once
#include "tfla_device.h"
#include "tfla_internal.h"

namespace tfla {

// SPLIT as in tile_kernel_bf16: 1 / 2 = the first / second D1-wide half of a contraction over 2 D1 columns (rows of
// X, Y and the state are 2 D1 apart); the first half stores its raw accumulators, the second adds them to its own.
// PAD: the caller's tensors end before the kernel's blocks do (TileArgs::out_T, out_ld, in_ld1); what lies past is zero.
template <int D1, int BD2, int NW, int MODE> struct TileShapeF32 {
    static constexpr int BC = 32, YS = D1 + Elem<float>::PAD, ZS = BC + Elem<float>::PAD;
    // Two stages of (Y tile, Z tile, column weights), one multiplied while the other is filled -- or, where two would
    // leave a CU with one workgroup (wide Y tiles), a single one behind a second barrier: the next tile waits in
    // registers meanwhile, and the other workgroups of the CU fill the gap.
    static constexpr int NSTG = 2 * (BC * YS + BD2 * ZS) * 4 <= 78 * 1024 ? 2 : 1;
    // LDS, in floats: Y tiles, Z tiles, column weights and their rounding remainders, per-row scalars, n_{k-1} (H)
    static constexpr int AT_Z = NSTG * BC * YS, AT_W = AT_Z + NSTG * BD2 * ZS, AT_WL = AT_W + NSTG * BC, AT_R = AT_WL + NSTG * BC,
                         AT_N = AT_R + NW * 32, FLOATS = AT_N + (MODE == MODE_H ? D1 : 0);
};

// One workgroup: output rows rbi and columns nb2 (block indices) of the chunk with the linear id wg.
template <int D1, int BD2, int NW, int MODE, int SPLIT, bool PAD>
__device__ __forceinline__ void tile_body_f32(const TileArgs& a, float* lds, int nb2, int rbi, unsigned wg) {
    using DT = float;
    using E = Elem<DT>;
    using frag = typename E::frag;
    using SH = TileShapeF32<D1, BD2, NW, MODE>;
    constexpr bool UPPER = (MODE & 1) != 0;
    constexpr int NT = NW * 64, BR = NW * 32, BC = SH::BC;
    constexpr int KS1 = D1 / 16, NB = BD2 / 32, NK = D1 / BC;
    constexpr int YS = SH::YS, ZS = SH::ZS, NSTG = SH::NSTG;
    constexpr int ld1 = SPLIT ? 2 * D1 : D1;    // row stride of the state's rows over the contraction index
    auto ldsY = reinterpret_cast<DT (*)[BC * YS]>(lds);
    auto ldsZ = reinterpret_cast<DT (*)[BD2 * ZS]>(lds + SH::AT_Z);
    auto ldsW = reinterpret_cast<float (*)[BC]>(lds + SH::AT_W);
    auto ldsWl = reinterpret_cast<float (*)[BC]>(lds + SH::AT_WL);  // rounding remainders of the column exponents (zeros when there are none)
    float* const ldsR = lds + SH::AT_R;
    float* const ldsN = lds + SH::AT_N;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
    const unsigned gy = (unsigned)a.L / (32 * NW);
    // later row blocks of a lower-triangular kernel (earlier ones of an upper one) have more column tiles: start them first
    const int rb = UPPER ? rbi : (int)gy - 1 - rbi;
    const int kc = wg % a.Nc, bh = wg / a.Nc;
    const long tbase = (long)bh * a.T + (long)kc * a.L;   // first step of the chunk
    const int r0 = rb * BR;                               // chunk-local first row of the workgroup
    const int wr0 = r0 + wave * 32;                       // ... of the wavefront
    const int d2 = a.d2;

    const DT* X = reinterpret_cast<const DT*>(a.X);
    // the caller's tensors: row strides, first step of the chunk, and (PAD) what is left of them from there on
    const int xld = PAD ? a.in_ld1 : ld1, zld = PAD ? a.out_ld : d2;
    const long tin = PAD ? (long)bh * a.out_T + (long)kc * a.L : tbase;
    const int steps_left = PAD ? a.out_T - kc * a.L : 0, cols1 = PAD ? a.in_cols1 : 0, cols2 = PAD ? a.out_ld - nb2 * BD2 : 0;
    const DT* Y = reinterpret_cast<const DT*>(a.Y) + tin * xld;
    const DT* Z = reinterpret_cast<const DT*>(a.Z) + tin * zld + (long)nb2 * BD2;
    // the state of the chunk is (d_hv, d_qk): contraction-contiguous for H and dV, contraction-major for dQ and dK
    constexpr bool STT = MODE == MODE_DQ || MODE == MODE_DK;
    const DT* St = reinterpret_cast<const DT*>(a.St) + (STT ? ((long)bh * a.Nc + kc) * ld1 * d2 + (long)nb2 * BD2
                                                            : (((long)bh * a.Nc + kc) * d2 + (long)nb2 * BD2) * ld1);
    const float* wcol = a.wcol + tbase;
    const float* wcol_lo = a.wcol_lo ? a.wcol_lo + tbase : nullptr;

    // X fragments of the wavefront's 32 rows (lane: row l32, k-group g)
    frag xf[KS1];
    {
        const DT* xr = X + (tin + wr0 + l32) * xld + 8 * g;
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) {
            if (!PAD || (wr0 + l32 < steps_left && 16 * ks + 8 * g < cols1)) xf[ks] = E::load(xr + 16 * ks);
            else xf[ks] = E::zero();
        }
    }
    if (MODE == MODE_H) {
        if (a.variant == 0)
            for (int i = tid; i < D1; i += NT) ldsN[i] = a.nstate[((long)bh * a.Nc + kc) * ld1 + i];
    }

    f32x16 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nb][v] = 0.0f;

    const int ct_lo = UPPER ? r0 / BC : 0;
    const int ct_hi = UPPER ? a.L / BC : (r0 + BR) / BC;

    typename std::conditional<STT, TrPrefetch<DT, BC, BD2, NT, false>, RowsPrefetch<DT, BD2, BC, NT>>::type ps;   // state slice [BD2][BC]
    auto load_state = [&](int j) {
        if constexpr (STT) ps.load(St + (long)j * BC * d2, d2, tid);
        else ps.load(St + j * BC, ld1, tid);
    };
    RowsPrefetch<DT, BC, D1, NT> py;           // Y tile       [BC][D1]
    TrPrefetch<DT, BC, BD2, NT, true> pz;      // Z tile       [BC][BD2] -> [BD2][BC]
    float pw = 0.0f, pwl = 0.0f;
    int buf = 0;
    auto other = [&]() { return NSTG == 2 ? buf ^ 1 : 0; };
    auto left = [&]() { if constexpr (NSTG == 1) __syncthreads(); };     // everyone has left the only stage

    // ---------------- inter-chunk part: acc = X_r St, BC columns of d1 per stage
    load_state(0);
    ps.store(ldsZ[0], ZS, tid);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        if (j + 1 < NK) {
            load_state(j + 1);
        } else {
            py.template load<PAD>(Y + (long)ct_lo * BC * xld, xld, tid, steps_left - ct_lo * BC, cols1);
            pz.template load<PAD>(Z + (long)ct_lo * BC * zld, zld, tid, steps_left - ct_lo * BC, cols2);
            if (tid < BC) { pw = wcol[ct_lo * BC + tid]; pwl = wcol_lo ? wcol_lo[ct_lo * BC + tid] : 0.0f; }
        }
        const DT* zb = ldsZ[buf];
#pragma unroll
        for (int ks = 0; ks < BC / 16; ++ks)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                acc[nb] = E::mma(xf[j * (BC / 16) + ks], E::load(zb + (nb * 32 + l32) * ZS + 16 * ks + 8 * g), acc[nb]);
        left();
        if (j + 1 < NK) {
            ps.store(ldsZ[other()], ZS, tid);
        } else {
            py.store(ldsY[other()], YS, tid);
            pz.store(ldsZ[other()], ZS, tid);
            if (tid < BC) { ldsW[other()][tid] = pw; ldsWl[other()][tid] = pwl; }
        }
        __syncthreads();
        buf = other();
    }
    {
        float sr[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) sr[v] = a.srow[tbase + wr0 + acc_row(v, g)];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nb][v] *= sr[v];
    }

    // mLSTMexp normaliser, inter-chunk part: srow_i * (q_i . n_{k-1}), one value per row
    float nrm = 0.0f;
    if (MODE == MODE_H) {
        if (a.variant == 0) {
            float dot = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) dot += E::frag_elem(xf[ks], e) * ldsN[16 * ks + 8 * g + e];
            dot += __shfl_xor(dot, 32, 64);
            nrm = dot * a.srow[tbase + wr0 + l32];
        }
    }

    // ---------------- intra-chunk part
    const float wr = a.wrow[tbase + wr0 + l32];
    const float wrl = a.wrow_lo ? a.wrow_lo[tbase + wr0 + l32] : 0.0f;
    float rowsum = 0.0f;
    for (int ct = ct_lo; ct < ct_hi; ++ct) {
        const int c0 = ct * BC;
        const bool more = ct + 1 < ct_hi;
        if (more) {
            py.template load<PAD>(Y + (long)(c0 + BC) * xld, xld, tid, steps_left - (c0 + BC), cols1);
            pz.template load<PAD>(Z + (long)(c0 + BC) * zld, zld, tid, steps_left - (c0 + BC), cols2);
            if (tid < BC) { pw = wcol[c0 + BC + tid]; pwl = wcol_lo ? wcol_lo[c0 + BC + tid] : 0.0f; }
        }
        const DT* yb = ldsY[buf];
        const DT* zb = ldsZ[buf];
        const float* wb = ldsW[buf];
        const float* wbl = ldsWl[buf];
#pragma unroll
        for (int st = 0; st < BC / 32; ++st) {
            const int cs = c0 + 32 * st;
            if (UPPER ? (cs + 31 < wr0) : (cs > wr0 + 31)) continue;      // fully masked for this wave
            const bool diag = UPPER ? (cs < wr0 + 31) : (cs + 31 > wr0);
            f32x16 s;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks)
                s = E::mma(E::load(yb + (32 * st + l32) * YS + 16 * ks + 8 * g), xf[ks], s);
            float p[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int cl = acc_row(v, g);
                // (rounded parts first: they nearly cancel, and their sum is exact in fp32)
                float w = fast_exp2((wr + wb[32 * st + cl]) + (wrl + wbl[32 * st + cl]));
                if (diag) {
                    const bool keep = UPPER ? (cs + cl >= wr0 + l32) : (cs + cl <= wr0 + l32);
                    w = keep ? w : 0.0f;
                }
                p[v] = s[v] * w;
                rowsum += p[v];
            }
            const frag p0 = E::pack(p), p1 = E::pack(p + 8);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const DT* zrow = zb + (nb * 32 + l32) * ZS + 32 * st + 8 * g;
                acc[nb] = E::mma(p0, E::load(zrow), acc[nb]);
                acc[nb] = E::mma(p1, E::load(zrow + 16), acc[nb]);
            }
        }
        left();
        if (more) {
            py.store(ldsY[other()], YS, tid);
            pz.store(ldsZ[other()], ZS, tid);
            if (tid < BC) { ldsW[other()][tid] = pw; ldsWl[other()][tid] = pwl; }
        }
        __syncthreads();
        buf = other();
    }

    // ---------------- epilogue
    float inv[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) inv[v] = 1.0f;
    if (MODE == MODE_H) {
        if (a.variant == 0) {
            rowsum += __shfl_xor(rowsum, 32, 64);
            nrm += rowsum;
        }
    }
    if constexpr (SPLIT == 1) {
        // first half: raw accumulators (and this half's share of the normaliser) for the second launch
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const long t = tbase + wr0 + acc_row(v, g);
                a.acc_out[t * d2 + (long)nb2 * BD2 + nb * 32 + l32] = acc[nb][v];
            }
        if (MODE == MODE_H && a.variant == 0 && g == 0 && nb2 == 0) a.nrm_out[tbase + wr0 + l32] = nrm;
        return;
    }
    if constexpr (SPLIT == 2) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const long t = tbase + wr0 + acc_row(v, g);
                acc[nb][v] += a.acc_in[t * d2 + (long)nb2 * BD2 + nb * 32 + l32];
            }
        if (MODE == MODE_H && a.variant == 0) nrm += a.nrm_in[tbase + wr0 + l32];
    }
    if (MODE == MODE_H) {
        if (a.variant == 0) {
            const long t = tbase + wr0 + l32;
            float den = fmaxf(fabsf(nrm), expf(-a.mout[t])) + a.eps;
            if (PAD && wr0 + l32 >= steps_left) den = 1.0f;     // (no q there: with eps = 0 and a large max state it would be 0)
            if (g == 0) {
                ldsR[wave * 32 + l32] = 1.0f / den;
                if (a.nout && nb2 == 0 && (!PAD || wr0 + l32 < steps_left)) a.nout[tin + wr0 + l32] = nrm;
                if (a.wrowB_out && nb2 == 0) {
                    if (a.wrowB_lo_out) {
                        const double w = (double)wr + (double)wrl - log2((double)den);
                        const float wh = (float)w;
                        a.wrowB_out[t] = wh;
                        a.wrowB_lo_out[t] = (float)(w - (double)wh);
                    } else {
                        a.wrowB_out[t] = a.wrow[t] - log2f(den);
                    }
                    a.sQ_out[t] = a.srow[t] / den;
                }
            }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 16; ++v) inv[v] = ldsR[wave * 32 + acc_row(v, g)];
        }
    }
    DT* Out = reinterpret_cast<DT*>(a.Out);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            // straight into the caller's tensor: its own row count and row length, true steps and columns only
            const int ts = wr0 + acc_row(v, g), col = nb * 32 + l32;
            if (!PAD || (ts < steps_left && col < cols2))
                Out[(tin + ts) * zld + nb2 * BD2 + col] = E::from_f32(acc[nb][v] * inv[v]);
        }
    if (MODE == MODE_DQ || MODE == MODE_DK) {
        const DT* W = reinterpret_cast<const DT*>(a.dotwith);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int ts = wr0 + acc_row(v, g);
            const long t = tbase + ts;
            float d = 0.0f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                if (!PAD || (ts < steps_left && nb * 32 + l32 < cols2))
                    d += acc[nb][v] * E::to_f32(W[(tin + ts) * zld + nb2 * BD2 + nb * 32 + l32]);
            d = half_sum(d);
            if (l32 == 0) a.dotpart[(long)nb2 * (long)a.dec_bh * a.T + t] = d;
        }
    }
}

template <int D1, int BD2, int NW, int MODE, int SPLIT = 0, bool PAD = false>
__global__ void __launch_bounds__(NW * 64) tile_kernel(TileArgs a) {
    __shared__ __attribute__((aligned(16))) float lds[TileShapeF32<D1, BD2, NW, MODE>::FLOATS];
    // one-dimensional launch (the number of workgroups can exceed what the y and z grid dimensions hold): linear id ->
    // (column block, row block, chunk, batch*head), column blocks fastest; the workgroups of one chunk (all column and
    // row blocks, which share K/V/state tiles) are neighbours on one XCD
    unsigned wg = xcd_remap(blockIdx.x, gridDim.x);
    const unsigned gx = (unsigned)a.d2 / BD2, gy = (unsigned)a.L / (32 * NW);
    const int nb2 = wg % gx; wg /= gx;
    const int rbi = wg % gy; wg /= gy;
    tile_body_f32<D1, BD2, NW, MODE, SPLIT, PAD>(a, lds, nb2, rbi, wg);
}

}  // namespace tfla
