// Intra-chunk tiled kernel (paper Sec. 3; App. C.3 Alg. 1 for H; App. C.4 for the three
// gradient kernels, with the parallel / loop dimensions of the paper's parallelisation table).
//
// One template covers the four kernels.  For a block of output rows r of one chunk:
//
//   out[r, :] = sum_{c causal} exp2(wrow[r] + wcol[c]) * (X_r . Y_c) * Z_c  +  srow[r] * (X_r St)
//
//   H   : X=Q  Y=K  Z=V   St=C_{k-1}^T        c <= r      (Alg. 1, both parts in one accumulator)
//   dV  : X=K  Y=Q  Z=dH  St=dC_k^T           c >= r
//   dQ  : X=dH Y=V  Z=K   St=C_{k-1}          c <= r
//   dK  : X=V  Y=dH Z=Q   St=dC_k             c >= r
//
// Differences from Alg. 1: the max state of every row is known from the gates alone (see the
// gate kernel), so the weights are final when they are formed -- no running maximum, no
// rescaling of the accumulator, and the inter-chunk product shares the accumulator and the
// register-resident X fragments with the intra-chunk loop for mLSTMexp as well.
//
// Work split: grid = (d2 / BD2, L / (32*NW), B*NH*Nc).  A wavefront owns 32 output rows and
// all BD2 columns of its workgroup; X_r stays in registers for the whole kernel; Y tiles
// (natural) and Z tiles (transposed, k-permuted) go through LDS and are shared by the
// waves.  The product (X_r . Y_c) is formed transposed (rows = c) so that its MFMA result is
// already laid out as the A operand of the second product.
#include "tfla_device.h"
#include "tfla_internal.h"
#include "tile_f32.h"
#include "tile_fast.h"
#include "tile_weights.h"

namespace tfla {

// ------------------------------------------------------------------------------------------
// what the bf16 kernels' decomposition of the linear workgroup id divides by
static void set_divisors(TileArgs& a, int BH, int gx, int gy) {
    auto log2_or_neg = [](int v) { return (v > 0 && (v & (v - 1)) == 0) ? __builtin_ctz((unsigned)v) : -1; };
    a.dec_bh = BH;
    a.dec_bpx = BH % 8 == 0 ? BH / 8 : 1;
    a.sh_gx = log2_or_neg(gx); a.sh_gy = log2_or_neg(gy);
    a.sh_bpx = log2_or_neg(a.dec_bpx); a.sh_nc = log2_or_neg(a.Nc);
}

// the weighted matrix of a mode into a.E (tile_weights.h); for H of mLSTMexp the row sums into a.nrm_out
template <int NW, int MODE>
static hipError_t launch_weights(TileArgs a, int BH, hipStream_t s) {
    const int gy = a.L / (32 * NW);
    set_divisors(a, BH, 1, gy);
    const dim3 grid((unsigned)((long)(gy * (gy + 1) / 2) * BH * a.Nc));
    if (a.out_T != a.T || a.in_ld1 != a.d1) hipLaunchKernelGGL((weights_kernel_bf16<NW, MODE, 1>), grid, dim3(64 * NW), 0, s, a);
    else hipLaunchKernelGGL((weights_kernel_bf16<NW, MODE, 0>), grid, dim3(64 * NW), 0, s, a);
    return hipGetLastError();
}

template <typename DT, int D1, int BD2, int NW, int MODE, int SPLIT = 0>
static hipError_t launch_tile_t(const TileArgs& a0, int BH, hipStream_t s) {
    TileArgs a = a0;
    dim3 grid((unsigned)((long)(a.d2 / BD2) * (a.L / (32 * NW)) * BH * a.Nc));
    // the caller's tensors may end before the kernels' blocks do
    const bool padded = a.out_T != a.T || a.out_ld != a.d2 || a.in_ld1 != (SPLIT ? 2 * D1 : D1);
    if constexpr (sizeof(DT) == 2) {
        set_divisors(a, BH, a.d2 / BD2, a.L / (32 * NW));
        // two workgroups per CU when the accumulator is narrow enough for 256 registers per lane
        constexpr int OCC = (BD2 <= 128 && D1 <= 256) ? 2 : 1;
        // dQ / dK share the weighted matrix E through memory only where the contraction that forms it is wide
        constexpr int NOE = D1 > 512 ? 2 : ((MODE == MODE_DQ || MODE == MODE_DK) && D1 <= TFLA_NOE_MAX_D1) ? 1 : 0;
        if constexpr (MODE == MODE_H && SPLIT == 0 && D1 <= 512 && BD2 <= 128) {
            // the layer output next to h~: whole rows in one workgroup, nothing padded (the entry point has checked)
            if (a.fz_y) {
                if (padded || a.d2 != BD2) return hipErrorInvalidValue;
                hipLaunchKernelGGL((tile_kernel_bf16<D1, BD2, NW, MODE, OCC, 0, 0, 0, 1>), grid, dim3(64 * NW), 0, s, a);
                return hipGetLastError();
            }
        }
        if (a.fz_y) return hipErrorInvalidValue;
        if (padded)
            hipLaunchKernelGGL((tile_kernel_bf16<D1, BD2, NW, MODE, OCC, SPLIT, NOE, 1>), grid, dim3(64 * NW), 0, s, a);
        else
            hipLaunchKernelGGL((tile_kernel_bf16<D1, BD2, NW, MODE, OCC, SPLIT, NOE, 0>), grid, dim3(64 * NW), 0, s, a);
    } else {
        a.dec_bh = BH;
        if (padded) hipLaunchKernelGGL((tile_kernel<D1, BD2, NW, MODE, SPLIT, true>), grid, dim3(64 * NW), 0, s, a);
        else hipLaunchKernelGGL((tile_kernel<D1, BD2, NW, MODE, SPLIT, false>), grid, dim3(64 * NW), 0, s, a);
    }
    return hipGetLastError();
}

template <typename DT, int D1, int MODE, int SPLIT = 0>
static hipError_t launch_tile_d1(const TileArgs& a, int BH, int bd2, hipStream_t s) {
    if (a.L % 128 == 0) {
        if constexpr (sizeof(DT) == 2 && D1 > 256) {   // see tile_bd2()
            if constexpr (D1 == 1024) {
                // 256 rows per workgroup, eight wavefronts: a third less to bring into LDS per result, which is what these
                // kernels wait for (7.5 TB/s with 128 rows).  16 heads of 1024, 4096 steps, chunk 256, H / dV / dQ / dK 268 / 239 /
                // 274 / 286 -> 224 / 209 / 232 / 239 us.  Forward + backward, 128 -> 256 rows, by the number of workgroups: 160 408 -> 342,
                // 192 479 -> 425, 256 529 -> 496, 416 875 -> 800, 448 896 -> 817, 512 949 -> 883, 528 1067 -> 1053, 576 1095 -> 1073, 640 1159 ->
                // 1115, 672 1285 -> 1189, 800 1516 -> 1460, 1024 1801 -> 1669; 1024 / 512 576 1340 -> 1335; 256 / 1024 640 1614 -> 1592; chunk 512 576
                // 1067 -> 991.  With a second round that is less than half full the two are within 2 % and which is faster
                // differs by shape: 288 636 -> 638 (1016 / 1000, 1000 steps 668 -> 679; chunk 768 615 -> 601), 320 649 -> 655 (689 -> 703; chunk 512
                // 635 -> 623), 384 741 -> 727 (800 -> 798; 1024 / 512 885 -> 890).  Those keep 128.
                const long wgs = (long)BH * a.T / 256 * (a.d2 / 256);
                if (bd2 == 256 && a.L % 256 == 0 && (wgs <= 256 || wgs > 384))
                    return launch_tile_t<DT, D1, 256, 8, MODE, SPLIT>(a, BH, s);
            }
            if (bd2 == 256) return launch_tile_t<DT, D1, 256, 4, MODE, SPLIT>(a, BH, s);
        }
        if (bd2 == 128) return launch_tile_t<DT, D1, 128, 4, MODE, SPLIT>(a, BH, s);
        if (bd2 == 64) return launch_tile_t<DT, D1, 64, 4, MODE, SPLIT>(a, BH, s);
        return hipErrorInvalidValue;    // the caller sized its buffers for a block width that is not built
    }
    if (bd2 == 128) return launch_tile_t<DT, D1, 128, 2, MODE, SPLIT>(a, BH, s);
    if (bd2 == 64) return launch_tile_t<DT, D1, 64, 2, MODE, SPLIT>(a, BH, s);
    return hipErrorInvalidValue;
}

template <typename DT, int MODE>
static hipError_t launch_tile_m(const TileArgs& a, int BH, int bd2, hipStream_t s) {
    switch (a.d1) {
        case 64: return launch_tile_d1<DT, 64, MODE>(a, BH, bd2, s);
        case 128: return launch_tile_d1<DT, 128, MODE>(a, BH, bd2, s);
        case 256: return launch_tile_d1<DT, 256, MODE>(a, BH, bd2, s);
        case 512:
            if (sizeof(DT) == 2) return launch_tile_d1<DT, (sizeof(DT) == 2 ? 512 : 64), MODE>(a, BH, bd2, s);
            break;
        default: break;
    }
    return hipErrorInvalidValue;
}

template <int MODE>
hipError_t launch_tile_mode(const TileArgs& a0, int BH, int dtype, hipStream_t s) {
    TileArgs a = a0;
    a.acc_in = nullptr; a.nrm_in = nullptr; a.acc_out = nullptr; a.nrm_out = nullptr;
    // Chunk order of each kernel of the sequence gates -> recurrence (first to last) -> H and reversed recurrence
    // (last to first) -> dV -> dQ -> dK, chosen by measurement (eight of the sixteen combinations on one box):
    // what matters is that H walks the chunks first to last, like the recurrence before it -- starting with the
    // states that were stored last (with non-temporal stores) costs 2 % of the step; among the gradient kernels
    // the differences are a few tenths of a percent, dK walking against dQ being the best.
#ifndef TFLA_KC_ORDER
#define TFLA_KC_ORDER 0x8   // bit m = 1: mode m walks the chunks last to first.  H, dV, dQ first to last, dK last to first
#endif
    a.kc_desc = ((TFLA_KC_ORDER) >> MODE) & 1;
    const int bd2 = tile_bd2(a.d1, a.d2, dtype, a.L, (long)BH * a.T);
    const bool nrm = MODE == MODE_H && a.variant == 0;
    if (dtype != 1) {
        if (a.d1 <= 256) return launch_tile_m<float, MODE>(a, BH, bd2, s);
        // fp32, d1 = 512: a wavefront's rows of X fill the register file at 256 fp32 columns, so the contraction runs
        // as two 256-wide launches that meet in fp32, like H of bf16 below in its last case
        if (a.d1 != 512 || !a.part_acc || (nrm && !a.part_nrm)) return hipErrorInvalidValue;
        TileArgs h = a;
        h.d1 = 256;
        h.acc_out = a.part_acc; h.nrm_out = a.part_nrm;
        hipError_t e = launch_tile_d1<float, 256, MODE, 1>(h, BH, bd2, s);
        if (e != hipSuccess) return e;
        h.acc_out = nullptr; h.nrm_out = nullptr;
        h.acc_in = a.part_acc; h.nrm_in = a.part_nrm;
        h.X = reinterpret_cast<const float*>(a.X) + 256;
        h.in_cols1 = a.in_cols1 - 256;
        h.Y = reinterpret_cast<const float*>(a.Y) + 256;
        h.St = reinterpret_cast<const float*>(a.St) + ((MODE == MODE_DQ || MODE == MODE_DK) ? (long)256 * a.d2 : 256);
        if (a.nstate) h.nstate = a.nstate + 256;
        return launch_tile_d1<float, 256, MODE, 2>(h, BH, bd2, s);
    }
    if (a.d1 <= 512) return launch_tile_m<bf16_t, MODE>(a, BH, bd2, s);
    // d1 = 1024: the kernels hold a workgroup's X rows in registers where they form the weighted matrix, which ends at 512
    // columns.  So a launch before them leaves the matrix in memory (dK reads what dQ's has left) and they read it.
    // 16 heads of 1024, 4096 steps, chunk 256, us per mode H / dV / dQ / dK, split contraction -> this: 454 / 461 / 501 / 421 ->
    // 312 / 280 / 316 / 249 (65 of the first three the weights), forward + backward 2758 -> 2087; chunk 128, 3000 steps of 8 heads
    // 1310 -> 1040; chunk 64, 2048 steps of 4 heads 848 -> 706.
    if (a.d1 != 1024) return hipErrorInvalidValue;
    constexpr bool STT = (MODE == MODE_DQ || MODE == MODE_DK);
    if (STT || weights_fit(a.L, a.d2, MODE)) {
        if (!STT) {
            if (!a.part_acc) return hipErrorInvalidValue;
            a.E = a.part_acc;
            if (MODE == MODE_H) a.nrm_in = a.nrm_out = reinterpret_cast<float*>(reinterpret_cast<char*>(a.part_acc) + (size_t)BH * a.T * a.L * 2);
        }
        if (!a.E) return hipErrorInvalidValue;
        if constexpr (MODE != MODE_DK) {
            hipError_t e = a.L % 128 == 0 ? launch_weights<4, MODE>(a, BH, s) : launch_weights<2, MODE>(a, BH, s);
            if (e != hipSuccess) return e;
        }
        return launch_tile_d1<bf16_t, 1024, MODE>(a, BH, bd2, s);
    }
    // H where d_hv is so narrow against the chunk that the matrix is larger than the memory for it: every term of the result is
    // linear in the products over d1 (the weights depend on the gates only), so the contraction runs as two launches over 512
    // columns each: the first leaves its unnormalised accumulators (and its share of the normaliser) in fp32, the second adds
    // them to its own before the epilogue.
    if constexpr (MODE == MODE_H) {
        if (!a.part_acc || (nrm && !a.part_nrm)) return hipErrorInvalidValue;
        TileArgs h = a;
        h.d1 = 512;
        h.acc_out = a.part_acc; h.nrm_out = a.part_nrm;
        hipError_t e = launch_tile_d1<bf16_t, 512, MODE, 1>(h, BH, bd2, s);
        if (e != hipSuccess) return e;
        h.acc_out = nullptr; h.nrm_out = nullptr;
        h.acc_in = a.part_acc; h.nrm_in = a.part_nrm;
        h.X = reinterpret_cast<const bf16_t*>(a.X) + 512;
        h.in_cols1 = a.in_cols1 - 512;
        h.Y = reinterpret_cast<const bf16_t*>(a.Y) + 512;
        h.St = reinterpret_cast<const bf16_t*>(a.St) + 512;
        // (n_{k-1} is stored as bf16 rows: 512 columns are 1024 bytes)
        if (a.nstate) h.nstate = reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.nstate) + 1024);
        return launch_tile_d1<bf16_t, 512, MODE, 2>(h, BH, bd2, s);
    }
    return hipErrorInvalidValue;
}

// One translation unit per (mode, element type) keeps compile times parallel: tile_inst.hip
// is compiled once for every TFLA_TILE_MODE.
template hipError_t launch_tile_mode<TFLA_TILE_MODE>(const TileArgs&, int, int, hipStream_t);

}  // namespace tfla
