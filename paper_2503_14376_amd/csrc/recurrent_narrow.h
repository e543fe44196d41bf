// The inter-chunk recurrent kernel (see recurrent.hip for what is computed) for problems with few state tiles, bf16.
//
//   state <- gbar_k * state + (rs (.) X_k)^T Y_k        (contraction over the rows of a chunk)
//
// A workgroup owns a 64 x 64 tile of the state for the whole sequence, half of what recurrent_kernel_bf16 takes, so that
// twice as many CUs work on one (batch, head), and consumes the sequence in pieces of BK rows.  With one workgroup per
// CU and no second one to hide its waits, the piece's chain of work is what counts, so its steps are spread over
// wavefronts of four kinds that run side by side between the workgroup barriers (one barrier per piece):
//   * 4 consumers: each keeps a quarter of the tile, 32 x 32, in MFMA accumulators and multiplies piece i into it; at a
//     chunk boundary it rounds the state into registers, applies the decay and stores the state behind the matrix
//     instructions;
//   * 4 producers bring the X part: into registers, four pieces ahead, and from there, multiplied by the row scales, into
//     the one of two LDS buffers that the consumers read next;
//   * 2 requesters bring the Y part: asynchronous global->LDS loads into a ring of NS stages, and the waits for them; and
//     the anchors of the forget-gate gradient scan, some pieces before they are needed.
// No wavefront waits for another one's memory operations but at the barrier; in recurrent_kernel_bf16, where the
// producers also request and the consumers also wait for Y, a piece takes 2300 clocks and a piece that opens a chunk
// 3400, whatever the load of the chip.
// Both operands are contracted over their row index, so both stay in their natural row-major layout in LDS and are read
// through the transposing LDS read.
// Measured, us per launch forward / reversed, 64 x 128 tiles of recurrent_kernel_bf16 against this as it first was, with two
// consumers: 8 heads 256 / 512, chunk 256, 8192 steps 97 / 96 -> 75 / 73; 16384 steps, chunk 512 151 / 150 -> 120 / 116; 32 heads
// of 128, 2048 steps, chunk 128 32 / 32 -> 26 / 24; 256 heads of 64, 2048 steps 37 / 32 -> 35 / 31.  With 16 heads 256 / 512, 512
// tiles for 256 CUs, it takes two rounds: 112 / 107 -> 142 / 135.
// What bounds it is the chain of a piece: with all memory operations left out it took 70 % of the time.  Clock stamps (8
// heads 256 / 512) gave 1540 clocks for a piece, 940 of them the consumers' reads and products on two of the four SIMDs,
// 600 more for one that opens a chunk (rounding the state), 800 more for the workgroups that keep the normaliser when one
// closes a chunk (eight sums over the wavefront) and 2900 more at an anchor, whose loads the consumers waited for.  With four
// consumers, those sums in registers and the anchors through LDS, forward + backward, us: 32 heads of 128, 2048 steps, chunk 128 104 ->
// 96; 4 heads of 512, 4096 steps 202 -> 195; 16 heads 96 / 192, batch 2, 3000 steps 194 -> 184; 8 heads 256 / 512, 8192 steps,
// chunk 64 652 -> 628, 256 416 -> 410; forward, 1000 steps, chunk 128 38.8 -> 35.7, 32768 steps, chunk 512 600 -> 587.
// More tiles than CUs (d_hv up to 64 has no other kernel).  In pieces of 64 rows two workgroups of the two-consumer form shared a
// CU, and two of this one do without the LDS for anchors (76 KB; loaded by the consumers then).  Forward + backward, us, two
// consumers / four without / four with it, which is one workgroup per CU: heads of 64, 2048 steps, chunk 64 320 tiles 388 / 388 / 383, 384
// 454 / 451 / 446, 512 601 / 590 / 588, 1024 1216 / 1207 / 1204, chunk 192 512 554 / 548 / 549; 1024 / 64, 1024 tiles 572 / 572 / 565; 256 / 64, 512 480 /
// 472 / 469; heads of 32, 1024 tiles 516 / 494 / 494; forward 258 / 245 / 246.
#pragma once
#include <type_traits>

#include "lds_tiles.h"
#include "tfla_internal.h"

namespace tfla {

// PAD: the caller's tensors end before the kernel's pieces and tiles do (RecArgs::T_in, d1_in, d2_in): loads past their
// end give zeros, and only what exists of the caller's states is read and written.
template <int BK, bool PAD>
__global__ void __launch_bounds__(640) recurrent_narrow_kernel_bf16(RecArgs a) {
    using E = Elem<bf16_t>;
    using frag = E::frag;
    constexpr int NC = 4, NP = 4, NR = 2;           // consumers, producers, requesters
    constexpr int BM = 64, BN = 64, KS = BK / 16;
    constexpr int XB = BK * BM * 2, YB = BK * BN * 2;
    constexpr int NS = BK == 64 ? 5 : 3;            // stages of the Y ring
    constexpr int NA = BK == 64 ? 4 : 2;            // buffers for anchors
    constexpr int D = 4;                            // pieces of X on their way in a producer's registers
    using DY = DmaTile<BK, BN, 64 * NR, SWZ_T>;
    constexpr int CPC = DY::N;                      // loads per requester and piece (Y)
    constexpr int NX = BK / 32;                     // 16-byte chunks of an X piece per producer lane
    constexpr int NST = 2;                          // state stores per consumer at a chunk boundary
    // pieces that the lines of X and Y are brought into L2 ahead (LinePrefetch).  8 heads 256 / 512, chunk 256, 8192 steps: 73.6 /
    // 73.0 us per launch forward / reversed without, 69.4 / 67.5 with 5, 69.9 / 68.3 with 6, 70.7 / 70.1 with 8; chunk 512 and
    // 16384 steps 120.8 / 117.3, 114.8 / 110.4, 112.5 / 107.2, 114.6 / 110.5.
    // Forward + backward in us, without -> with: 16 sharers, 128 / 512, 8192 steps, chunk 256 326 -> 317, 4096 steps,
    // chunk 64 376 -> 373; 8 heads of 256, 4096 steps, chunk 64 218 -> 217, 16 heads, 8192 steps, chunk 256 426 -> 425; 32 sharers,
    // 512 / 256, chunk 64 372 -> 363, 256 / 512, 8192 steps, chunk 64 688 -> 681.
    constexpr int AHEAD = 6;

    __shared__ __attribute__((aligned(1024))) char smemY[NS * YB];
    __shared__ __attribute__((aligned(1024))) char smemX[2 * XB];
    __shared__ __attribute__((aligned(256))) float ldsG[4096];                  // gbar of every chunk
    __shared__ __attribute__((aligned(256))) float ldsPf[NR][64];               // where the prefetches go
    __shared__ __attribute__((aligned(256))) float ldsNx[2][NP][BM];            // column sums of scaled X, per producer
    __shared__ __attribute__((aligned(1024))) char ldsAnc[NA * BM * BN * 4];    // anchors of the tile
    __shared__ float ldsDot[NC];                                                // a consumer's part of an anchor's product

    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool producer = wave >= NC && wave < NC + NP, requester = wave >= NC + NP;
    const int wc = wave >= NC ? wave - NC : wave;   // index among consumers or producers
    const unsigned nwg = gridDim.x * gridDim.y * gridDim.z;
    unsigned wg = xcd_remap(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), nwg);
    // readfirstlane: tell the compiler these are wave-uniform, so that everything derived from them
    // lives in scalar registers
    const int bx = __builtin_amdgcn_readfirstlane((int)(wg % gridDim.x)); wg /= gridDim.x;
    const int by = __builtin_amdgcn_readfirstlane((int)(wg % gridDim.y));
    const int bh = __builtin_amdgcn_readfirstlane((int)(wg / gridDim.y));
    const int n0 = bx * BN, m0 = by * BM;
    const int PPC = a.L / BK, P = a.Nc * PPC;
    // the normaliser vector n (one value per state row) is kept by the workgroups bx == 0:
    // lane l of the first producer owns row m0 + l
    const bool with_n = (a.nst != nullptr) && bx == 0;
    // the caller's tensors: row strides, steps per (batch, head), and (PAD) columns from this tile's first on
    const int xld = PAD ? a.d1_in : a.d1, yld = PAD ? a.d2_in : a.d2, tld = PAD ? a.T_in : a.T;
    const int xcols = PAD ? a.d1_in - m0 : 0, ycols = PAD ? a.d2_in - n0 : 0;
    // Pieces are taken in order and the addresses advance incrementally; when the recurrence runs backwards the chunks
    // are visited last to first, rows inside a chunk still ascending, so the step at a chunk's end is BK - 2 L rows.
    const long row0 = a.reverse ? (long)(a.Nc - 1) * a.L : 0;
    const int step_rows = BK, wrap_rows = a.reverse ? BK - 2 * a.L : BK;

    if (requester) {
        // =============================== requester ===========================================
        __builtin_amdgcn_s_setprio(3);
        const int rtid = tid - 64 * (NC + NP);
        const int rw = __builtin_amdgcn_readfirstlane(rtid >> 6);
        DY dy; dy.init(yld, rtid);
        if constexpr (PAD) dy.bound_columns(ycols, rtid);
        const bf16_t* yreq = reinterpret_cast<const bf16_t*>(a.Y) + ((long)bh * tld + row0) * yld + n0;
        int yleft = PAD ? a.T_in - (int)row0 : 0;
        int lsub = 0, lslot = 0;
        const uint32_t ya = lds_addr(smemY);
        uint32_t lst = ya;
        // requester 0 prefetches X, requester 1 Y
        LinePrefetch<BK, AHEAD> pf;
        if constexpr (!PAD) {       // (tensors that end inside a piece are left as they were: 8 heads, 1000 steps with layer 39.4 us without, 40.3 with)
            pf.init(rw == 0 ? a.X : a.Y, bh, rw == 0 ? xld : yld, tld, rw == 0 ? a.d1 : a.d2, (int)(gridDim.x * gridDim.y),
                    by * (int)gridDim.x + bx, P, row0, lane, lds_addr(ldsPf) + 256u * rw);
            if (pf.on)
                for (int p = 0; p < AHEAD; ++p) pf.advance(PPC, step_rows, wrap_rows);
        }
        auto request = [&]() {
            if constexpr (PAD) dy.template issue_bounded<true>(yreq, bounded_bytes(yleft, ycols, 2 * yld), BN, lst, rtid);
            else dy.issue(yreq, lst, rtid);
            const bool wrap = ++lsub == PPC;
            const int dr = wrap ? wrap_rows : step_rows;
            yreq += (long)dr * yld; yleft -= dr;
            if (wrap) lsub = 0;
            if (++lslot == NS) { lslot = 0; lst = ya; } else lst += YB;
            if (pf.on) { pf.issue(); pf.advance(PPC, step_rows, wrap_rows); }
        };
        constexpr int AH = NS - 2;      // pieces younger than the awaited one
        static_assert(AH * (CPC + 1) + 1 + (AH + 1) / 2 * 8 <= 63, "the counter holds the pieces on their way");
        // Anchors (reversed launch, see the consumers): the 16 KB of the next one are requested DA pieces before the piece that
        // opens its chunk, ahead of that iteration's piece, so that the wait for the latter covers them.  Anchors are at least
        // two pieces apart (anchor_chunks()), so that the consumers have left the buffer NA anchors ago.
        constexpr int DA = NS == 3 ? 3 : AH + 1, ACH = BM * BN * 4 / 1024 / NR;         // pieces; wave loads per requester and anchor
        static_assert(DA >= AH + 1 && DA <= NS - 1 + (NS == 3) && 2 * NA >= DA + 1, "an anchor lands in time, into a free buffer");
        int anc_left = a.anc_in ? (a.Nc - 1) / a.anc_G : 0, anc_buf = 0;
        unsigned anc_recent = 0;                                                        // anchors of the last AH iterations, a bit each
        const int kb0 = anc_left * a.anc_G;
        int anc_at = (a.Nc - kb0) * PPC - DA;
        const int nslot = (a.Nc + a.anc_G - 1) / a.anc_G;
        const float* asrc = a.anc_in + ((long)bh * nslot + anc_left) * a.d1 * a.d2 + (long)(by * (int)gridDim.x + bx) * (BM * BN) + rw * ACH * 256;
        auto request_anchor = [&]() {
            const uint32_t dst = lds_addr(ldsAnc) + (uint32_t)(anc_buf * (BM * BN * 4) + rw * ACH * 1024);
#pragma unroll
            for (int q = 0; q < ACH; ++q) dma16_nt(asrc + q * 256, (uint32_t)lane * 16u, dst + q * 1024);
            asrc -= (long)a.d1 * a.d2;
            anc_buf = (anc_buf + 1) % NA; --anc_left; anc_at += a.anc_G * PPC;
        };
        while (anc_left && anc_at < 0) request_anchor();
        for (int p = 0; p < NS - 1 && p < P; ++p) request();
        auto await = [&](int younger) {     // pieces requested after the awaited one
            // (the prefetch that was issued right behind the awaited piece need not have landed)
            if (younger >= AH) {
                if (pf.on) wait_vmcnt<AH * (CPC + 1) + 1>();
                else wait_vmcnt<AH * CPC>();
            } else wait_vmcnt_dyn(pf.on ? younger * (CPC + 1) + 1 : younger * CPC);
        };
        await((P < NS - 1 ? P : NS - 1) - 1);
        int i = 0;
        for (; i < P; ++i) {
            barrier_nofence();
            // piece i + NS - 1 goes into the stage of piece i - 1, which every consumer has left; piece i + 1 must have landed
            // before the next barrier
            anc_recent = (anc_recent << 1) & ((1u << AH) - 1);
            if (anc_left && i == anc_at) { request_anchor(); anc_recent |= 1; }
            if (i + NS - 1 < P) {
                request();
                if (anc_recent) wait_vmcnt_dyn(__builtin_popcount(anc_recent) * ACH + (pf.on ? AH * (CPC + 1) + 1 : AH * CPC));
                else await(AH);
            }
            else await(P - 2 - i > 0 ? P - 2 - i : 0);
        }
        for (; i % D != 0; ++i) barrier_nofence();      // (the producers' iterations come in groups of D)
        wait_vmcnt<0>();                                // (nothing is on its way into LDS when the workgroup ends)
    } else if (producer) {
        // =============================== producers ===========================================
        __builtin_amdgcn_s_setprio(3);
        const bool n_owner = with_n && wc == 0;
        // gbar of the whole sequence, for the consumers' chunk boundaries (and the normaliser)
        for (int k = wc * 64 + lane; k < a.Nc; k += NP * 64) ldsG[k] = a.gbar[(long)bh * a.Nc + k];
        float nacc = (n_owner && a.n0 && (!PAD || lane < xcols)) ? a.n0[(long)bh * xld + m0 + lane] : 0.0f;
        float nsum[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) nsum[e] = 0.0f;
        // this lane's part of a piece: eight columns of NX consecutive rows, whose scales are one load
        const int pr = (wc * 8 + (lane >> 3)) * NX, pc = lane & 7;
        const bf16_t* xreq = reinterpret_cast<const bf16_t*>(a.X) + ((long)bh * tld + row0) * xld + m0;
        const float* rsreq = a.rs + (long)bh * a.T + row0;
        int xleft = PAD ? a.T_in - (int)row0 : 0;      // steps of the sequence from the next piece's first on
        uint32_t xoff[NX];                             // byte offsets of its chunks within a piece
#pragma unroll
        for (int j = 0; j < NX; ++j) xoff[j] = (uint32_t)((pr + j) * xld + pc * 8) * 2u;
        typedef float scales __attribute__((ext_vector_type(NX)));
        u32x4 xv[D][NX];
        scales xs[D];
        int lsub = 0, left = P;                        // pieces still to request
        // (past the last piece it is requested again: the number of loads in flight is then the same in every
        // iteration, which is what the compiler's waits are computed from)
        auto request_chunk = [&](int slot, int j) {
            const char* src = reinterpret_cast<const char*>(xreq) + xoff[j];
            if (PAD) xv[slot][j] = (pr + j < xleft && pc * 8 < xcols) ? *reinterpret_cast<const u32x4*>(src) : u32x4{0u, 0u, 0u, 0u};
            else xv[slot][j] = *reinterpret_cast<const u32x4*>(src);
        };
        auto request_scales = [&](int slot) { xs[slot] = *reinterpret_cast<const scales*>(reinterpret_cast<const char*>(rsreq) + (uint32_t)pr * 4u); };
        auto advance = [&]() {
            // (selected, not branched over: with branches the compiler's waits come out as if the pieces had been
            // requested in another order)
            const int more = --left > 0 ? 1 : 0;
            const bool wrap = lsub + 1 == PPC;
            const int dr = more * (wrap ? wrap_rows : step_rows);
            xreq += (long)dr * xld; rsreq += dr; xleft -= dr;
            lsub = wrap ? 0 : lsub + 1;
        };
        auto request = [&](int slot) {
            request_scales(slot);
#pragma unroll
            for (int j = 0; j < NX; ++j) request_chunk(slot, j);
            advance();
        };
        // Scale the piece in `slot` (of chunk step `stp`, last of its chunk if `closes`) into LDS buffer `buf`; a piece is
        // requested into the registers of `rslot` on the way (none if negative).
        auto rescale = [&](int slot, int buf, int stp, bool closes, int rslot) {
            if (rslot >= 0) request_scales(rslot);
            char* xt = smemX + buf * XB;
#pragma unroll
            for (int j = 0; j < NX; ++j) {
                if (rslot >= 0) request_chunk(rslot, j);
                const float sc = xs[slot][j];
                u32x4 w = xv[slot][j];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const float lo = bf16_lo_to_f32(w[d]) * sc, hi = bf16_hi_to_f32(w[d]) * sc;
                    if (with_n) { nsum[2 * d] += lo; nsum[2 * d + 1] += hi; }
                    w[d] = pack_bf16x2(lo, hi);
                }
                const int r = pr + j;
                *reinterpret_cast<u32x4*>(xt + r * (BM * 2) + ((pc ^ swz_mask<SWZ_T, BM / 8>(r)) * 16)) = w;
            }
            if (rslot >= 0) advance();
            // the piece that closes a chunk also closes the chunk's column sums
            if (with_n && closes) {
                // Lanes that hold the same eight columns differ in lane bits 3 to 5.  Two values at a time are added over a
                // bit, each half of the lanes keeping one of the sums: in the end lane l holds column 8 (l & 7) + e.
                // (Eight sums in every lane are 24 shuffles.)
                const auto over32 = [](float x, float y) {
                    const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
                    return __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);
                };
                const auto over16 = [](float x, float y) {
                    const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y), false, false);
                    return __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);
                };
                float r[4], t[2];
#pragma unroll
                for (int k = 0; k < 4; ++k) r[k] = over32(nsum[k], nsum[k + 4]);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    t[k] = over16(r[k], r[k + 2]);
                    t[k] += dpp_move<0x128>(t[k]);      // row_ror:8
                }
                const int e = ((lane >> 3) & 1) + 2 * ((lane >> 4) & 1) + 4 * g;
                ldsNx[stp & 1][wc][8 * (lane & 7) + e] = (lane & 8) ? t[1] : t[0];
#pragma unroll
                for (int e = 0; e < 8; ++e) nsum[e] = 0.0f;
            }
        };
#pragma unroll
        for (int p = 0; p < D; ++p) request(p);
        rescale(0, 0, 0, PPC == 1, -1);

        // Iteration i (consumers multiply piece i from buffer i & 1): scale piece i + 1 into the other buffer, which the
        // consumers left at the barrier, and request piece i + D into the registers of piece i.
        // (sub, step) describe piece i.
        int sub = 0, step = 0;
        for (int i0 = 0; i0 < P; i0 += D) {
            // (whole groups of D: leaving in the middle would again spoil the compiler's waits)
#pragma unroll
            for (int dd = 0; dd < D; ++dd) {
                const int i = i0 + dd;
                // the scaled chunks must have landed before the barrier hands them over
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                barrier_nofence();
                // normaliser vector: piece i closes its chunk, whose column sums every producer has just
                // published; emit n before that chunk, then apply the chunk
                if (n_owner && sub == PPC - 1 && i < P) {
                    const int kc = a.reverse ? a.Nc - 1 - step : step;
                    // n before this chunk leaves as two bf16 rows of d1: the rounded value and the rounding
                    // remainder (together good to 2^-17), the form in which the parallel kernel feeds it to the
                    // matrix unit next to the state
                    // (stores the compiler does not count: known ones on a path that is not always taken would make its
                    // waits for the X pieces stricter by more than a piece; unknown ones make them at most two loads
                    // stricter)
                    const uint16_t* np = reinterpret_cast<const uint16_t*>(a.nst) + ((long)bh * a.Nc + kc) * 2 * a.d1 + m0;
                    const uint32_t nhi = bf16_bits_rne(nacc);
                    store16_uncounted(np, (uint32_t)lane * 2u, nhi);
                    store16_uncounted(np + a.d1, (uint32_t)lane * 2u, bf16_bits_rne(nacc - bf16_lo_to_f32(nhi)));
                    float s = 0.0f;
#pragma unroll
                    for (int w = 0; w < NP; ++w) s += ldsNx[step & 1][w][lane];
                    nacc = ldsG[kc] * nacc + s;
                }
                int sub1 = sub + 1, step1 = step;
                if (sub1 == PPC) { sub1 = 0; ++step1; }
                rescale((dd + 1) % D, (i + 1) & 1, step1, sub1 == PPC - 1, dd);
                sub = sub1; step = step1;
            }
        }
        if (n_owner && a.nfinal && (!PAD || lane < xcols)) a.nfinal[(long)bh * xld + m0 + lane] = nacc;
    } else {
        // =============================== consumers ===========================================
        const int wn = wc & 1, wm = wc >> 1;        // column block, row block
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = m0 + wm * 32 + acc_row(v, g);
            const int n = n0 + wn * 32 + l32;
            const bool there = !PAD || (m < a.d1_in && n < a.d2_in);
            acc[v] = (a.S0 && there) ? a.S0[((long)bh * xld + m) * yld + n] : 0.0f;
        }
        // make the compiler wait for these plain loads here rather than inside the loop, where its
        // wait would also cover the state stores in flight
#pragma unroll
        for (int v = 0; v < 16; ++v) asm volatile("" : "+v"(acc[v]));
        const uint32_t aoff = TFragReader<BM>::offset_of(lane, 8, wm);      // LDS byte offsets of this wave's blocks
        const uint32_t boff = TFragReader<BN>::offset_of(lane, 8, wn);
        int sub = 0, step = 0, slot = 0;
        int kc = a.reverse ? a.Nc - 1 : 0;
        // the next anchor boundary (see below): the multiples of anc_G strictly between 0 and Nc, upwards or downwards
        int kb_next = a.reverse ? ((a.Nc - 1) / a.anc_G) * a.anc_G : (a.anc_G < a.Nc ? a.anc_G : 0);
        if (kb_next == 0) kb_next = -1;
        char* const st0p = reinterpret_cast<char*>(a.stT) + (((long)bh * a.Nc * a.d2 + n0 + wn * 32 + (lane & 15)) * a.d1 + m0 + wm * 32 + 16 * ((lane >> 4) & 1) + 8 * g) * 2;
        const long stchunk = (long)a.d1 * a.d2 * 2;

        int abuf = 0;               // where the next anchor lies
        long dot_at = -1;           // where the product whose parts are in ldsDot goes
        int i = 0;
        for (; i < P; ++i) {
            // (the fragment reads of the piece before have left the buffers that are refilled from here on)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            barrier_nofence();
            if (dot_at >= 0) {       // (an anchor never belongs to the last piece)
                if (wm == 0 && lane == 0) a.anc_part[dot_at] = ldsDot[wn] + ldsDot[2 + wn];
                dot_at = -1;
            }
            const char* xt = smemX + (i & 1) * XB;
            const char* yt = smemY + slot * YB;
            // Chunk boundary: the state before this chunk's update leaves, then it decays.  It is rounded into registers here
            // and stored behind the matrix instructions, where the memory pipeline's queue holds nothing up.
            // Registers 4 j .. 4 j + 3 are four consecutive state rows of this lane's column; the two halves of the
            // wavefront hold the two halves of every eight.  Exchanged between the halves, a lane has eight consecutive
            // ones, 16 bytes of the transposed state's row, and the halves 32 contiguous bytes.
            u32x4 stw[NST];
            const bool boundary = sub == 0;
            const int kst = kc;
            if (boundary) {
                const float gb = ldsG[kc];
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    const uint32_t a0 = pack_bf16x2(acc[4 * j], acc[4 * j + 1]), a1 = pack_bf16x2(acc[4 * j + 2], acc[4 * j + 3]);
                    const uint32_t b0 = pack_bf16x2(acc[4 * j + 4], acc[4 * j + 5]), b1 = pack_bf16x2(acc[4 * j + 6], acc[4 * j + 7]);
                    const auto s0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
                    stw[j / 2] = u32x4{s0[0], s1[0], s0[1], s1[1]};
                }
                // ... and between the rows of 16 lanes: 64 contiguous bytes of 16 rows per store
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const auto t = __builtin_amdgcn_permlane16_swap(stw[0][d], stw[1][d], false, false);
                    stw[0][d] = t[0]; stw[1][d] = t[1];
                }
                // Boundaries between the blocks of the forget-gate gradient scan (the state here is the one between
                // chunks kb - 1 and kb): the forward launch leaves an fp32 copy of its accumulators, the reversed
                // launch multiplies that copy with its own and leaves the partial inner product.
                if (a.anc || a.anc_in) {
                    const int kb = a.reverse ? kc + 1 : kc;
                    if (kb == kb_next) {
                        kb_next += a.reverse ? -a.anc_G : a.anc_G;
                        if (kb_next >= a.Nc || kb_next <= 0) kb_next = -1;     // (no more)
                        const long per = (long)a.d1 * a.d2;
                        const int nslot = (a.Nc + a.anc_G - 1) / a.anc_G;
                        const int part = (by * (int)gridDim.x + bx) * 2 + wn;
                        const long off = ((long)bh * nslot + kb / a.anc_G) * per + ((long)(part * 8 + wm * 4) * 64 + lane) * 4;
                        if (a.anc) {
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const f32x4 w = {acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]};
                                // (read again only by the reversed launch, much later: non-temporal)
                                __builtin_nontemporal_store(w, reinterpret_cast<f32x4*>(a.anc + off + (long)j * 256));
                            }
                        }
                        if (a.anc_in) {
                            const char* ap = ldsAnc + abuf * (BM * BN * 4) + (wn * 8 + wm * 4) * 1024 + lane * 16;
                            f32x4 c[4];
#pragma unroll
                            for (int j = 0; j < 4; ++j) c[j] = *reinterpret_cast<const f32x4*>(ap + j * 1024);
                            abuf = (abuf + 1) % NA;
                            float dot = 0.0f;
#pragma unroll
                            for (int j = 0; j < 4; ++j)
#pragma unroll
                                for (int e = 0; e < 4; ++e) dot += acc[4 * j + e] * c[j][e];
                            dot = wave_sum(dot);
                            if (lane == 0) ldsDot[wc] = dot;
                            dot_at = ((long)bh * nslot + kb / a.anc_G) * (gridDim.x * gridDim.y * 2) + part;
                        }
                    }
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] *= gb;
            }
            // LDS reads run two k steps ahead of the matrix instructions
            frag af[KS], bfr[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                af[ks].v = TFragReader<BM>::load_at(xt, aoff, 16 * ks, 16 * ks + 4);
                bfr[ks].v = TFragReader<BN>::load_at(yt, boff, 16 * ks, 16 * ks + 4);
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = E::mma(af[ks], bfr[ks], acc);
            constexpr int PF = 2;
#pragma unroll
            for (int q = 0; q < PF; ++q) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int q = 0; q < KS - PF; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            }
#pragma unroll
            for (int q = 0; q < PF; ++q) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (boundary && a.stT) {
                char* gdst = st0p + (long)kst * stchunk;
#pragma unroll
                for (int q = 0; q < NST; ++q) *reinterpret_cast<u32x4*>(gdst + (long)q * 16 * a.d1 * 2) = stw[q];
            }
            if (++sub == PPC) { sub = 0; ++step; kc += a.reverse ? -1 : 1; }
            if (++slot == NS) slot = 0;
        }
        for (; i % D != 0; ++i) barrier_nofence();      // (the producers' iterations come in groups of D)
        if (a.Sfinal || a.Sfinal2) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int m = m0 + wm * 32 + acc_row(v, g);
                const int n = n0 + wn * 32 + l32;
                const bool there = !PAD || (m < a.d1_in && n < a.d2_in);
                if (a.Sfinal && there) a.Sfinal[((long)bh * xld + m) * yld + n] = acc[v];
                if (a.Sfinal2) a.Sfinal2[((long)bh * a.d1 + m) * a.d2 + n] = acc[v];
            }
        }
    }
}

}  // namespace tfla
