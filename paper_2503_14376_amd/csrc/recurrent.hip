// Inter-chunk recurrent kernel (paper Sec. 3 "recurrent kernel"; App. B.2 inter-chunk
// recurrence; App. B.3 recurrence of delta C).  Sequential over chunks, parallel over
// (batch*head) and over BM x BN tiles of the d1 x d2 state.
//
//   state <- gbar_k * state + (rs (.) X_k)^T Y_k
//
// Forward:  X = K, Y = V, rs = a-bar, state = C;  backward: X = Q, Y = delta H,
// rs = b-bar * qscale / h_denom, state = delta C, chunks visited last to first.  The state
// before each update is written (in the element type of X/Y) to slot k in the layout the tiled
// kernels read: stT[k] = state^T (d2 x d1).
#include "tfla_device.h"
#include "tfla_internal.h"
#include "recurrent_fast.h"
#include "recurrent_narrow.h"

namespace tfla {

// fp32 kernel.  Pieces of BK rows of X (scaled) and Y go through registers into LDS in their own row-major layout: the
// fp32 matrix instructions take one value per lane and k, so the fragments are read from it as they are.  D pieces are on
// their way in registers.  What bounds it: the matrix instructions, 1024 clocks per piece and wavefront in one chain, and
// the staging around them in the same wavefronts.  (With both operands transposed on the way, a dword per load, and waits
// that drained the pieces at every branch: 16 heads 128 x 256, 1024 steps, chunk 64 52 us per launch, then 43.)
// PAD: the caller's tensors end before the pieces and tiles do (RecArgs::T_in, d1_in, d2_in); what lies past is zero.
template <int MI, int NI, bool PAD>
__global__ void __launch_bounds__(256) recurrent_kernel_f32(RecArgs a) {
    constexpr int BM = 64 * MI, BN = 64 * NI, NT = 256, BK = 32, D = 4;
    constexpr int LX = BM + 4, LY = BN + 4;
    __shared__ __attribute__((aligned(16))) float ldsX[2][BK * LX];
    __shared__ __attribute__((aligned(16))) float ldsY[2][BK * LY];
    __shared__ float ldsG[4096];                // gbar of every chunk

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    // XCD-aware decomposition: all state tiles of one (batch, head) share K/V and sit on one XCD
    const unsigned nwg = gridDim.x * gridDim.y * gridDim.z;
    unsigned wg = xcd_remap(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), nwg);
    const int bx = wg % gridDim.x; wg /= gridDim.x;
    const int by = wg % gridDim.y; const int bh = wg / gridDim.y;
    const int n0 = bx * BN, m0 = by * BM;
    // the caller's tensors: row strides, and (PAD) what exists of them from this tile's first column on
    const int xld = PAD ? a.d1_in : a.d1, yld = PAD ? a.d2_in : a.d2, tld = PAD ? a.T_in : a.T;
    const int xcols = PAD ? a.d1_in - m0 : 0, ycols = PAD ? a.d2_in - n0 : 0;
    const float* X = reinterpret_cast<const float*>(a.X) + (long)bh * tld * xld + m0;
    const float* Y = reinterpret_cast<const float*>(a.Y) + (long)bh * tld * yld + n0;
    const float* rs = a.rs + (long)bh * a.T;
    const bool with_n = (a.nst != nullptr) && bx == 0;

    for (int k = tid; k < a.Nc; k += NT) ldsG[k] = a.gbar[(long)bh * a.Nc + k];
    f32x16 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + wm * 32 * MI + 32 * mi + acc_row(v, g);
                const int n = n0 + wn * 32 * NI + 32 * ni + l32;
                const bool there = !PAD || (m < a.d1_in && n < a.d2_in);
                acc[mi][ni][v] = (a.S0 && there) ? a.S0[((long)bh * xld + m) * yld + n] : 0.0f;
            }
        }
    float nacc = 0.0f;
    if (with_n && tid < BM && a.n0 && (!PAD || tid < xcols)) nacc = a.n0[(long)bh * xld + m0 + tid];

    // The sequence is consumed as P pieces of BK rows; piece i belongs to chunk step i / PPC.  Past the last piece it is
    // requested again, and the loop runs whole groups of D pieces: the compiler's waits for the pieces on their way are
    // exact only if every path has the same loads.
    const int PPC = a.L / BK, P = a.Nc * PPC;
    using PX = RowsPrefetch<float, BK, BM, NT>;
    using PY = RowsPrefetch<float, BK, BN, NT>;
    PX px[D];
    PY py[D];
    float prs[D][PX::N];
    auto request = [&](int slot, int i0) {
        const int i = i0 < P ? i0 : P - 1;
        const int stepc = i / PPC, kc = a.reverse ? a.Nc - 1 - stepc : stepc;
        const long tr = (long)kc * a.L + (long)(i - stepc * PPC) * BK;
#pragma unroll
        for (int j = 0; j < PX::N; ++j) prs[slot][j] = rs[tr + (tid + j * NT) / PX::CPR];
        px[slot].template load<PAD>(X + tr * xld, xld, tid, tld - (int)tr, xcols);
        py[slot].template load<PAD>(Y + tr * yld, yld, tid, tld - (int)tr, ycols);
    };
    auto stage = [&](int slot, int buf) {
#pragma unroll
        for (int j = 0; j < PX::N; ++j) {
            f32x4 w = __builtin_bit_cast(f32x4, px[slot].r[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] *= prs[slot][j];
            px[slot].r[j] = __builtin_bit_cast(u32x4, w);
        }
        px[slot].store(ldsX[buf], LX, tid);
        py[slot].store(ldsY[buf], LY, tid);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(d, d);
    stage(0, 0);
    __syncthreads();

    for (int i0 = 0; i0 < P; i0 += D) {
#pragma unroll
        for (int dd = 0; dd < D; ++dd) {
            const int i = i0 + dd;
            // ---- request piece i + D into the registers of piece i, stage piece i + 1 into the other LDS buffer
            request(dd, i + D);
            stage((dd + 1) % D, (i + 1) & 1);
            const float* xb = ldsX[i & 1] + wm * 32 * MI + l32;
            const float* yb = ldsY[i & 1] + wn * 32 * NI + l32;
            if (i < P) {
                // ---- chunk boundary: emit the state before this chunk's update, then decay
                if (i % PPC == 0) {
                    const int stepc = i / PPC;
                    const int kc = a.reverse ? a.Nc - 1 - stepc : stepc;
                    const long slot = (long)bh * a.Nc + kc;
                    const float gb = ldsG[kc];
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) {
                            const int n = n0 + wn * 32 * NI + 32 * ni + l32;
                            if (a.stT) {
                                // registers 4j..4j+3 hold four consecutive m: one packed store each
                                float* dst = reinterpret_cast<float*>(a.stT) + slot * a.d1 * a.d2;
#pragma unroll
                                for (int j = 0; j < 4; ++j) {
                                    const int m = m0 + wm * 32 * MI + 32 * mi + acc_row(4 * j, g);
                                    store4(dst + (long)n * a.d1 + m, acc[mi][ni][4 * j], acc[mi][ni][4 * j + 1],
                                           acc[mi][ni][4 * j + 2], acc[mi][ni][4 * j + 3]);
                                }
                            }
#pragma unroll
                            for (int v = 0; v < 16; ++v) acc[mi][ni][v] *= gb;
                        }
                    if (with_n && tid < BM) a.nst[slot * a.d1 + m0 + tid] = nacc;
                    nacc *= gb;
                }
                // ---- multiply piece i
#pragma unroll
                for (int k = 0; k < BK; k += 2) {
                    float af[MI], bf[NI];
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) af[mi] = xb[(k + g) * LX + 32 * mi];
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) bf[ni] = yb[(k + g) * LY + 32 * ni];
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[mi], bf[ni], acc[mi][ni], 0, 0, 0);
                }
                if (with_n && tid < BM) {
                    // n += column sums of the staged (a-bar (.) K) piece, from the same rounded values
                    float sacc = 0.0f;
#pragma unroll
                    for (int c = 0; c < BK; ++c) sacc += ldsX[i & 1][c * LX + tid];
                    nacc += sacc;
                }
            }
            __syncthreads();
        }
    }
    // ---- final state
    if (a.Sfinal || a.Sfinal2) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = m0 + wm * 32 * MI + 32 * mi + acc_row(v, g);
                    const int n = n0 + wn * 32 * NI + 32 * ni + l32;
                    const bool there = !PAD || (m < a.d1_in && n < a.d2_in);
                    if (a.Sfinal && there) a.Sfinal[((long)bh * xld + m) * yld + n] = acc[mi][ni][v];
                    if (a.Sfinal2) a.Sfinal2[((long)bh * a.d1 + m) * a.d2 + n] = acc[mi][ni][v];
                }
    }
    if (with_n && tid < BM && a.nfinal && (!PAD || tid < xcols)) a.nfinal[(long)bh * xld + m0 + tid] = nacc;
}

// The same for fewer state tiles: 64 x 32 tiles, twice as many workgroups, and the rows of a piece split between two
// wavefronts, so that a piece is 512 clocks of matrix instructions instead of 1024.  The state is the sum of the two
// wavefronts' accumulators; at a chunk boundary both leave them in LDS, and everyone stores the sum one piece later, in whole
// rows of 256 bytes.  The column sums for the normaliser are spread over the four wavefronts in the same way.
// LX = 96: the two half-waves read rows of X that are one apart, and lie in different banks.
template <bool PAD>
__global__ void __launch_bounds__(256) recurrent_split_kernel_f32(RecArgs a) {
    constexpr int BM = 64, BN = 32, NT = 256, BK = 32, D = 4, LX = 96, LY = 32, LS = BM + 4;
    __shared__ __attribute__((aligned(16))) float ldsX[2][BK * LX];
    __shared__ __attribute__((aligned(16))) float ldsY[2][BK * LY];
    __shared__ __attribute__((aligned(16))) float ldsS[2][BN * LS];     // the two parts of the state, (n, m)
    __shared__ float ldsN[4][BM];
    __shared__ float ldsG[4096];                // gbar of every chunk

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, g = lane >> 5;
    const int wm = wave >> 1, kh = wave & 1;    // rows of the tile, half of a piece
    // XCD-aware decomposition: all state tiles of one (batch, head) share K/V and sit on one XCD
    const unsigned nwg = gridDim.x * gridDim.y * gridDim.z;
    unsigned wg = xcd_remap(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), nwg);
    const int bx = wg % gridDim.x; wg /= gridDim.x;
    const int by = wg % gridDim.y; const int bh = wg / gridDim.y;
    const int n0 = bx * BN, m0 = by * BM;
    const int xld = PAD ? a.d1_in : a.d1, yld = PAD ? a.d2_in : a.d2, tld = PAD ? a.T_in : a.T;
    const int xcols = PAD ? a.d1_in - m0 : 0, ycols = PAD ? a.d2_in - n0 : 0;
    const float* X = reinterpret_cast<const float*>(a.X) + (long)bh * tld * xld + m0;
    const float* Y = reinterpret_cast<const float*>(a.Y) + (long)bh * tld * yld + n0;
    const float* rs = a.rs + (long)bh * a.T;
    const bool with_n = (a.nst != nullptr) && bx == 0;

    for (int k = tid; k < a.Nc; k += NT) ldsG[k] = a.gbar[(long)bh * a.Nc + k];
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int m = m0 + wm * 32 + acc_row(v, g), n = n0 + l32;
        const bool there = kh == 0 && (!PAD || (m < a.d1_in && n < a.d2_in));
        acc[v] = (a.S0 && there) ? a.S0[((long)bh * xld + m) * yld + n] : 0.0f;
    }
    float nacc = (with_n && a.n0 && wave == 0 && (!PAD || lane < xcols)) ? a.n0[(long)bh * xld + m0 + lane] : 0.0f;

    // (pieces as in the kernel above)
    const int PPC = a.L / BK, P = a.Nc * PPC;
    using PX = RowsPrefetch<float, BK, BM, NT>;
    using PY = RowsPrefetch<float, BK, BN, NT>;
    PX px[D];
    PY py[D];
    float prs[D][PX::N];
    auto request = [&](int slot, int i0) {
        const int i = i0 < P ? i0 : P - 1;
        const int stepc = i / PPC, kc = a.reverse ? a.Nc - 1 - stepc : stepc;
        const long tr = (long)kc * a.L + (long)(i - stepc * PPC) * BK;
#pragma unroll
        for (int j = 0; j < PX::N; ++j) prs[slot][j] = rs[tr + (tid + j * NT) / PX::CPR];
        px[slot].template load<PAD>(X + tr * xld, xld, tid, tld - (int)tr, xcols);
        py[slot].template load<PAD>(Y + tr * yld, yld, tid, tld - (int)tr, ycols);
    };
    auto stage = [&](int slot, int buf) {
#pragma unroll
        for (int j = 0; j < PX::N; ++j) {
            f32x4 w = __builtin_bit_cast(f32x4, px[slot].r[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] *= prs[slot][j];
            px[slot].r[j] = __builtin_bit_cast(u32x4, w);
        }
        px[slot].store(ldsX[buf], LX, tid);
        py[slot].store(ldsY[buf], LY, tid);
    };
    // this wavefront's part of the state into LDS: registers 4 j .. 4 j + 3 are four consecutive m of column n
    auto publish = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            store4(&ldsS[kh][l32 * LS + wm * 32 + acc_row(4 * j, g)], acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]);
        if (with_n) ldsN[wave][lane] = nacc;
    };
    // the sum of both parts to slot kc (one piece after publish())
    auto emit = [&](int kc) {
        const long slot = (long)bh * a.Nc + kc;
        if (a.stT) {
            float* dst = reinterpret_cast<float*>(a.stT) + slot * a.d1 * a.d2 + (long)n0 * a.d1 + m0;
#pragma unroll
            for (int h = 0; h < BN * BM / 4 / NT; ++h) {
                const int idx = tid + h * NT, n = idx >> 4, m = 4 * (idx & 15);
                const f32x4 w = *reinterpret_cast<const f32x4*>(&ldsS[0][n * LS + m]) + *reinterpret_cast<const f32x4*>(&ldsS[1][n * LS + m]);
                *reinterpret_cast<f32x4*>(dst + (long)n * a.d1 + m) = w;
            }
        }
        if (with_n && tid < BM) a.nst[slot * a.d1 + m0 + tid] = (ldsN[0][tid] + ldsN[1][tid]) + (ldsN[2][tid] + ldsN[3][tid]);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(d, d);
    stage(0, 0);
    __syncthreads();

    int sub = 0, kc = a.reverse ? a.Nc - 1 : 0;         // piece i within its chunk, its chunk
    for (int i0 = 0; i0 < P; i0 += D) {
#pragma unroll
        for (int dd = 0; dd < D; ++dd) {
            const int i = i0 + dd;
            // ---- request piece i + D into the registers of piece i, stage piece i + 1 into the other LDS buffer
            request(dd, i + D);
            stage((dd + 1) % D, (i + 1) & 1);
            const float* xb = ldsX[i & 1] + kh * 16 * LX + wm * 32 + l32;
            const float* yb = ldsY[i & 1] + kh * 16 * LY + l32;
            if (i < P) {
                float af[8], bf[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) { af[k] = xb[(2 * k + g) * LX]; bf[k] = yb[(2 * k + g) * LY]; }
                // ---- chunk boundary: the state before this chunk's update leaves, then it decays
                if (sub == 0) {
                    publish();
                    const float gb = ldsG[kc];
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[v] *= gb;
                    nacc *= gb;
                }
                // ---- multiply piece i
#pragma unroll
                for (int k = 0; k < 8; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[k], bf[k], acc, 0, 0, 0);
                if (sub == 1) emit(kc);         // (a chunk has at least two pieces)
                if (with_n) {
                    // n += column sums of the staged (a-bar (.) K) piece, from the same rounded values
                    float sacc = 0.0f;
#pragma unroll
                    for (int c = 0; c < BK / 4; ++c) sacc += ldsX[i & 1][(wave * (BK / 4) + c) * LX + lane];
                    nacc += sacc;
                }
                if (++sub == PPC) { sub = 0; kc += a.reverse ? -1 : 1; }
            }
            __syncthreads();
        }
    }
    // ---- final state
    publish();
    __syncthreads();
    if (a.Sfinal || a.Sfinal2) {
#pragma unroll
        for (int h = 0; h < BM * BN / NT; ++h) {
            const int idx = tid + h * NT, mi = idx / BN, ni = idx % BN, m = m0 + mi, n = n0 + ni;
            const float w = ldsS[0][ni * LS + mi] + ldsS[1][ni * LS + mi];
            const bool there = !PAD || (m < a.d1_in && n < a.d2_in);
            if (a.Sfinal && there) a.Sfinal[((long)bh * xld + m) * yld + n] = w;
            if (a.Sfinal2) a.Sfinal2[((long)bh * a.d1 + m) * a.d2 + n] = w;
        }
    }
    if (with_n && tid < BM && a.nfinal && (!PAD || tid < xcols))
        a.nfinal[(long)bh * xld + m0 + tid] = (ldsN[0][tid] + ldsN[1][tid]) + (ldsN[2][tid] + ldsN[3][tid]);
}

static hipError_t launch_rec_split_f32(const RecArgs& a, int BH, hipStream_t s) {
    const dim3 grid(a.d2 / 32, a.d1 / 64, BH);
    if (a.padded()) hipLaunchKernelGGL((recurrent_split_kernel_f32<true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((recurrent_split_kernel_f32<false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int MI, int NI>
static hipError_t launch_rec_f32(const RecArgs& a, int BH, hipStream_t s) {
    dim3 grid(a.d2 / (64 * NI), a.d1 / (64 * MI), BH);
    if (a.padded()) hipLaunchKernelGGL((recurrent_kernel_f32<MI, NI, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((recurrent_kernel_f32<MI, NI, false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <bool PAD>
static hipError_t launch_rec_bf16(const RecArgs& a, int BH, hipStream_t s) {
    // 64 x 128 state tiles where they are whole and 64 x 64 ones would not fit the 256 CUs in one round (see
    // recurrent_narrow.h for both sides); pieces of 128 rows (half as many barriers) where the chunk size allows.
    // Many tiles: 128 x 256 ones (in pieces of 64 rows), which fetch half as many bytes of X and Y per state value; a
    // round of workgroups of them lasts about 8/3 rounds of the others.  Forward + backward in us, 64 x 128 -> 128 x 256,
    // by the number of 128 x 256 tiles (heads of 512, 2048 steps, chunk 256): 128 346 -> 361, 160 485 -> 457, 192 503 -> 481, 224 639 -> 587,
    // 256 656 -> 597, 288 808 -> 816, 320 838 -> 842, 352 973 -> 937, 512 1278 -> 1173, 576 1449 -> 1406; 256 / 512, 256 tiles
    // 732 -> 670; heads of 256, 256 tiles 782 -> 746; 16 heads of 1024, 4096 steps 2040 -> 1797 (launches 471 -> 342).
    // The chunk does not move the line, also where every piece opens one.  Chunk 64: 136 700 -> 664, 192 854 -> 823, 256 1157 -> 1040,
    // 768 3524 -> 3129, 256 / 512, 160 757 -> 727, 128 / 256, 256 648 -> 630, heads of 1024, 512 2027 -> 1775; 128: 192 523 -> 514, 256 699 -> 641; 192:
    // 192 747 -> 694, 256 992 -> 892; 512: 192 603 -> 548, 256 742 -> 686.
    const long tall_tiles = a.d1 % 128 == 0 && a.d2 % 256 == 0 ? (long)BH * (a.d1 / 128) * (a.d2 / 256) : 0;
    if (tall_tiles > 0 && 8 * ((tall_tiles + 255) / 256) <= 3 * ((4 * tall_tiles + 255) / 256)) {
        hipLaunchKernelGGL((recurrent_kernel_bf16<8, 64, PAD, 128, 4>), dim3(a.d2 / 256, a.d1 / 128, BH), dim3(768), 0, s, a);
        return hipGetLastError();
    }
    const bool narrow = a.d2 % 128 != 0 || (long)BH * (a.d1 / 64) * (a.d2 / 64) <= 256;
    const bool wide_pieces = a.L % 128 == 0;
    const dim3 grid(a.d2 / (narrow ? 64 : 128), a.d1 / 64, BH), block(512);
    if (narrow) {
        if (wide_pieces) hipLaunchKernelGGL((recurrent_narrow_kernel_bf16<128, PAD>), grid, dim3(640), 0, s, a);
        else hipLaunchKernelGGL((recurrent_narrow_kernel_bf16<64, PAD>), grid, dim3(640), 0, s, a);
    } else {
        if (wide_pieces) hipLaunchKernelGGL((recurrent_kernel_bf16<4, 128, PAD>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((recurrent_kernel_bf16<4, 64, PAD>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_recurrent(const RecArgs& a, int BH, int dtype, hipStream_t s) {
    if (dtype == 1) {
        return a.padded() ? launch_rec_bf16<true>(a, BH, s) : launch_rec_bf16<false>(a, BH, s);
    }
    // fp32: 64 x 32 tiles with the rows of a piece split between two wavefronts while 64 x 64 ones would not give every CU one
    // (us per launch forward / reversed, 64 x 64 -> split: 1 head of 64, 256 steps 15.5 / 12.7 -> 12.1 / 10.9; 16 heads of
    // 128 / 256, 1024 steps, chunk 64 43 / 37 -> 33 / 29; 128 heads of 32, 1024 steps 44 / 37 -> 32 / 29; at exactly 256 tiles, 64 heads
    // of 128, 4096 steps 180 / 155 -> 151 / 131; at 512, 32 heads of 256 225 / 203 -> 254 / 229 and 8 of 512, 512 steps 38 / 32 ->
    // 45 / 41); beyond, 128 x 128 tiles when they still fill the chip, else 64 x 64
    if ((long)BH * (a.d1 / 64) * (a.d2 / 64) <= 256) return launch_rec_split_f32(a, BH, s);
    const bool big_ok = (a.d1 % 128 == 0) && (a.d2 % 128 == 0);
    const long wg_big = (long)BH * (a.d1 / 128) * (a.d2 / 128);
    const bool big = big_ok && wg_big >= 192;
    return big ? launch_rec_f32<2, 2>(a, BH, s) : launch_rec_f32<1, 1>(a, BH, s);
}

}  // namespace tfla

#ifdef TFLA_TIMELINE
extern "C" __attribute__((visibility("default"))) int tfla_debug_rec_timeline(unsigned long long* host, size_t n) {
    return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(tfla::tfla_rec_timeline), n * sizeof(unsigned long long));
}
#endif
