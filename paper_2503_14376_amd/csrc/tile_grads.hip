// dV, dQ and dK of every chunk in one launch.
//
// The three gradient kernels of a chunk read the same tensors (K, Q and dH in all of them, V and the states in two), and
// where dQ and dK form their weighted matrix each for itself (tile_shares_E()) none waits for another.  One after another,
// each streams its operands from memory again; side by side on one XCD they find them in its L2: 64 heads of 64, batch 4,
// 2048 steps: 316 MB fetched, 302 MB of operands counted once, 788 MB as each part reads them (the chunks that are under way on an XCD at a time have 1.5 MB of them
// there, 4 MB at heads of 256).  Forward + backward, three launches -> one: that shape with its layer 415 -> 374 us, 32 heads
// of 128 345 -> 305, 16 heads of 256 440 -> 413, 16 heads of 96 / 192 and 3000 steps 234 -> 209, one sequence of 777 steps
// and 8 heads of 64 / 128, where two launches fewer count, 71 -> 52.  fp32: one head of 64 and 256 steps 87 -> 60 us (three
// launches of 11 - 16 us on four CUs -> one of 15), 16 heads of 128 / 256 and 1024 steps 243 -> 229.
// Linear workgroup id: (chunk of a head, row block, {column blocks of dV, of dQ, of dK}), the last fastest.  Every part is
// the body of its own kernel (tile_fast.h, tile_f32.h) in the same LDS; registers and LDS are those of the widest.  In bf16 that
// still leaves two workgroups per CU; in fp32 most of the wide ones take more than 256 registers and run one wavefront per SIMD,
// as the kernels of their own do there, and 40 of the 68 spill scalar registers (up to 179, the ragged and 128-wide ones most):
// the argument blocks of three parts are live at once.
//
// Compiled once per TFLA_GRADS_DQK (kernel width of q and k); a unit holds the kernels of that width only.
#include "tfla_device.h"
#include "tfla_internal.h"
#include "tile_f32.h"
#include "tile_fast.h"

#ifndef TFLA_GRADS_DQK
#error "compile with -DTFLA_GRADS_DQK=<64, 128 or 256>"
#endif

namespace tfla {

struct GradTileArgs { TileArgs dv, dq, dk; };

template <int DQK, int DHV, int NW, int PAD>
__global__ void __launch_bounds__(NW * 64, 2) grads_kernel_bf16(GradTileArgs a) {
    constexpr int BV = DHV >= 128 ? 128 : 64, BQ = DQK >= 128 ? 128 : 64;
    using SV = TileShape<DQK, BV, NW, MODE_DV, 2, 0, 0, 0>;
    using SQ = TileShape<DHV, BQ, NW, MODE_DQ, 2, 0, 1, 0>;
    using SK = TileShape<DHV, BQ, NW, MODE_DK, 2, 0, 1, 0>;
    constexpr int M = SV::BYTES > SQ::BYTES ? SV::BYTES : SQ::BYTES, BYTES = M > SK::BYTES ? M : SK::BYTES;
    __shared__ __attribute__((aligned(1024))) char smem[BYTES];
    auto pieces = [&](auto s) {
        using S = decltype(s);
        return TileLds{smem, smem + S::AT_E, reinterpret_cast<float*>(smem + S::AT_W), reinterpret_cast<float*>(smem + S::AT_S),
                       reinterpret_cast<float*>(smem + S::AT_WR), reinterpret_cast<float*>(smem + S::AT_M), reinterpret_cast<float*>(smem + S::AT_N)};
    };
    constexpr unsigned GV = DHV / BV, GQ = DQK / BQ;
    unsigned wg = xcd_remap(blockIdx.x, gridDim.x), rem;
    wg = tile_divmod(wg, GV + 2 * GQ, -1, rem);
    const int part = __builtin_amdgcn_readfirstlane((int)rem);
    wg = tile_divmod(wg, (unsigned)a.dv.L / (32 * NW), a.dv.sh_gy, rem);
    const int rbi = __builtin_amdgcn_readfirstlane((int)rem);
    if (part < (int)GV) tile_body_bf16<DQK, BV, NW, MODE_DV, 2, 0, 0, PAD, 0, false>(a.dv, pieces(SV{}), part, rbi, wg);
    else if (part < (int)(GV + GQ)) tile_body_bf16<DHV, BQ, NW, MODE_DQ, 2, 0, 1, PAD, 0, false>(a.dq, pieces(SQ{}), part - (int)GV, rbi, wg);
    else tile_body_bf16<DHV, BQ, NW, MODE_DK, 2, 0, 1, PAD, 0, false>(a.dk, pieces(SK{}), part - (int)(GV + GQ), rbi, wg);
}

template <int DQK, int DHV, int NW, bool WIDE, bool PAD>
__global__ void __launch_bounds__(NW * 64) grads_kernel_f32(GradTileArgs a) {
    constexpr int BV = WIDE && DHV >= 128 ? 128 : 64, BQ = WIDE && DQK >= 128 ? 128 : 64;
    constexpr int FV = TileShapeF32<DQK, BV, NW, MODE_DV>::FLOATS, FQ = TileShapeF32<DHV, BQ, NW, MODE_DQ>::FLOATS;
    __shared__ __attribute__((aligned(16))) float lds[FV > FQ ? FV : FQ];
    constexpr unsigned GV = DHV / BV, GQ = DQK / BQ;
    unsigned wg = xcd_remap(blockIdx.x, gridDim.x);
    const int part = wg % (GV + 2 * GQ); wg /= GV + 2 * GQ;
    const unsigned gy = (unsigned)a.dv.L / (32 * NW);
    const int rbi = wg % gy; wg /= gy;
    if (part < (int)GV) tile_body_f32<DQK, BV, NW, MODE_DV, 0, PAD>(a.dv, lds, part, rbi, wg);
    else if (part < (int)(GV + GQ)) tile_body_f32<DHV, BQ, NW, MODE_DQ, 0, PAD>(a.dq, lds, part - (int)GV, rbi, wg);
    else tile_body_f32<DHV, BQ, NW, MODE_DK, 0, PAD>(a.dk, lds, part - (int)(GV + GQ), rbi, wg);
}

template <int DQK, int DHV, int NW, bool WIDE>
static hipError_t launch_grads_f32(const GradTileArgs& a, dim3 grid, bool padded, hipStream_t s) {
    if (padded) hipLaunchKernelGGL((grads_kernel_f32<DQK, DHV, NW, WIDE, true>), grid, dim3(64 * NW), 0, s, a);
    else hipLaunchKernelGGL((grads_kernel_f32<DQK, DHV, NW, WIDE, false>), grid, dim3(64 * NW), 0, s, a);
    return hipGetLastError();
}

template <int DQK, int DHV, int NW>
static hipError_t launch_grads_t(GradTileArgs& a, int BH, int dtype, hipStream_t s) {
    const int wide = dtype == 1 || grads_f32_wide(DQK, DHV, (long)BH * a.dv.T) ? 128 : 64;
    const int BV = DHV < wide ? DHV : wide, BQ = DQK < wide ? DQK : wide;
    auto log2_or_neg = [](int v) { return (v > 0 && (v & (v - 1)) == 0) ? __builtin_ctz((unsigned)v) : -1; };
    TileArgs* const m[3] = {&a.dv, &a.dq, &a.dk};
    for (TileArgs* t : m) {
        t->kc_desc = 0;
        t->dec_bh = BH;
        t->dec_bpx = BH % 8 == 0 ? BH / 8 : 1;
        t->sh_gx = -1; t->sh_gy = log2_or_neg(t->L / (32 * NW));
        t->sh_bpx = log2_or_neg(t->dec_bpx); t->sh_nc = log2_or_neg(t->Nc);
    }
    const dim3 grid((unsigned)((long)(DHV / BV + 2 * (DQK / BQ)) * (a.dv.L / (32 * NW)) * BH * a.dv.Nc));
    const bool padded = a.dv.out_T != a.dv.T || a.dv.out_ld != DHV || a.dq.out_ld != DQK;
    if (dtype != 1) {
        if constexpr (DQK >= 128 || DHV >= 128) {
            if (wide == 128) return launch_grads_f32<DQK, DHV, NW, true>(a, grid, padded, s);
        }
        return launch_grads_f32<DQK, DHV, NW, false>(a, grid, padded, s);
    }
    if (padded) hipLaunchKernelGGL((grads_kernel_bf16<DQK, DHV, NW, 1>), grid, dim3(64 * NW), 0, s, a);
    else hipLaunchKernelGGL((grads_kernel_bf16<DQK, DHV, NW, 0>), grid, dim3(64 * NW), 0, s, a);
    return hipGetLastError();
}

template <int DQK>
hipError_t launch_tile_grads(const TileArgs& dv, const TileArgs& dq, const TileArgs& dk, int BH, int dtype, hipStream_t s) {
    GradTileArgs a{dv, dq, dk};
    const bool w4 = dv.L % 128 == 0;
    switch (dv.d2) {
        case 64: return w4 ? launch_grads_t<DQK, 64, 4>(a, BH, dtype, s) : launch_grads_t<DQK, 64, 2>(a, BH, dtype, s);
        case 128: return w4 ? launch_grads_t<DQK, 128, 4>(a, BH, dtype, s) : launch_grads_t<DQK, 128, 2>(a, BH, dtype, s);
        case 256: return w4 ? launch_grads_t<DQK, 256, 4>(a, BH, dtype, s) : launch_grads_t<DQK, 256, 2>(a, BH, dtype, s);
        default: return hipErrorInvalidValue;
    }
}
template hipError_t launch_tile_grads<TFLA_GRADS_DQK>(const TileArgs&, const TileArgs&, const TileArgs&, int, int, hipStream_t);

}  // namespace tfla
