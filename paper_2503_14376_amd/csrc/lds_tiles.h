// bf16 tiles in LDS for gfx950: filled asynchronously by global->LDS loads (no registers, no
// VALU work), read either as k-contiguous MFMA fragments (ds_read_b128) or, when the
// contraction index is the tile's row index, through the transposing LDS read
// (ds_read_b64_tr_b16).  Tiles are stored unpadded in their natural row-major layout; bank
// conflicts are avoided by XOR-swizzling the 16-byte chunks of each row.
//
// global->LDS load (global_load_lds_dwordx4): every lane supplies its own 16-byte global
// address; the 64 results land at consecutive 16-byte slots from a wave-uniform LDS address.
//
// transposing read (ds_read_b64_tr_b16), per group of 16 lanes: source lane j supplies the
// address of four consecutive 16-bit elements; result lane i receives, for e = 0..3, element
// (i & 3) of source lane 4e + (i >> 2).  With source lane j pointing at row k0 + (j >> 2),
// columns n0 + 4 (j & 3) .. +3 of a row-major tile, result lane i holds rows k0..k0+3 of
// column n0 + i: four consecutive contraction indices for the lane's own column, which is
// what an MFMA operand needs.
#pragma once
#include "tfla_device.h"

namespace tfla {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

enum { SWZ_K = 0, SWZ_T = 1 };   // tile read by k-contiguous fragments / by transposing reads

// XOR mask (in 16-byte chunks) applied to the chunk index of row r; CPR = chunks per row.
template <int KIND, int CPR> __device__ __forceinline__ int swz_mask(int r) {
    if (KIND == SWZ_K) {
        if (CPR >= 16) return r & 15;
        if (CPR == 8) return (r >> 1) & 7;
        return (r >> 2) & 3;
    }
    static_assert(KIND == SWZ_K || CPR >= 8, "a transposed tile has at least 64 columns: the mask moves a chunk by four");
    if (CPR >= 16) return 4 * (r & 3);
    return 4 * ((r >> 1) & 1);
}

// 32-bit LDS address of a __shared__ object
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// One global->LDS load of 64 x 16 bytes: lane l copies 16 bytes from gbase + voff(l) to LDS
// address lds_uniform + 16 * l.  Issued through inline assembly so that the compiler's
// wait-count insertion does not serialise later LDS reads of *other* pipeline stages behind
// it; the kernels order these loads themselves with wait_vmcnt + barrier.
__device__ __forceinline__ void dma16(const void* gbase_uniform, uint32_t voff, uint32_t lds_uniform) {
    const uint32_t la = __builtin_amdgcn_readfirstlane(lds_uniform);
    const uint64_t gb = (uint64_t)(uintptr_t)gbase_uniform;
    // readfirstlane returns a signed int: go through uint32_t so the low half is not sign-extended
    const uint32_t glo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gb);
    const uint32_t ghi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gb >> 32));
    const uint64_t gu = (uint64_t)glo | ((uint64_t)ghi << 32);
    // s_nop 4: the hardware needs 5 wait states between a write of an SGPR (the base address, M0) and
    // a vector-memory instruction that reads it; the compiler's hazard recogniser cannot see inside
    // the asm, so the distance is guaranteed here
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(la), "v"(voff), "s"(gu) : "memory", "m0");
}

// The same load without the "memory" clobber: the compiler may move ordinary LDS reads and MFMAs
// across it (it stays ordered with the kernels' barriers and waits, which are volatile asm too).
// For loads that are issued between matrix instructions into a stage nobody reads in that phase.
__device__ __forceinline__ void dma16_free(const void* gbase_uniform, uint32_t voff, uint32_t lds_uniform) {
    const uint32_t la = __builtin_amdgcn_readfirstlane(lds_uniform);
    const uint64_t gb = (uint64_t)(uintptr_t)gbase_uniform;
    const uint32_t glo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gb);
    const uint32_t ghi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gb >> 32));
    const uint64_t gu = (uint64_t)glo | ((uint64_t)ghi << 32);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(la), "v"(voff), "s"(gu) : "m0");
}

// The two loads above with the non-temporal hint: for operands that exactly one workgroup of the launch reads,
// so that they do not displace what several workgroups share from the caches.
__device__ __forceinline__ void dma16_nt(const void* gbase_uniform, uint32_t voff, uint32_t lds_uniform) {
    const uint32_t la = __builtin_amdgcn_readfirstlane(lds_uniform);
    const uint64_t gb = (uint64_t)(uintptr_t)gbase_uniform;
    const uint32_t glo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gb);
    const uint32_t ghi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gb >> 32));
    const uint64_t gu = (uint64_t)glo | ((uint64_t)ghi << 32);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :: "s"(la), "v"(voff), "s"(gu) : "memory", "m0");
}
__device__ __forceinline__ void dma16_free_nt(const void* gbase_uniform, uint32_t voff, uint32_t lds_uniform) {
    const uint32_t la = __builtin_amdgcn_readfirstlane(lds_uniform);
    const uint64_t gb = (uint64_t)(uintptr_t)gbase_uniform;
    const uint32_t glo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gb);
    const uint32_t ghi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gb >> 32));
    const uint64_t gu = (uint64_t)glo | ((uint64_t)ghi << 32);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :: "s"(la), "v"(voff), "s"(gu) : "m0");
}

// The same load through a buffer descriptor: lanes whose offset lies at or beyond `bytes` (measured from gbase) read
// nothing and leave zeros in LDS.  For operands that end before the tile does: the steps past the end of a sequence and
// the columns past a head dimension are filled with zeros on the way instead of being copied into padded buffers first.
// CLOBBER: ordered with the surrounding memory accesses like dma16, else free like dma16_free.
// (The non-temporal hint of dma16_nt for rows and dot operands that one workgroup alone reads is not worth a variant here:
// forward + backward of ragged problems 1.5 % faster to 2.7 % slower with it, heads of 128 and of 96 / 192.)
template <bool CLOBBER>
__device__ __forceinline__ void dma16_bounded(const void* gbase_uniform, uint32_t bytes, uint32_t voff, uint32_t lds_uniform) {
    const uint32_t la = __builtin_amdgcn_readfirstlane(lds_uniform);
    const uint64_t gb = (uint64_t)(uintptr_t)gbase_uniform;
    u32x4 rsrc;
    rsrc[0] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gb);
    rsrc[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gb >> 32)) & 0xffffu;   // stride 0: a raw buffer
    rsrc[2] = (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes);
    rsrc[3] = 0x00020000u;                                                                    // 32-bit data format
    if constexpr (CLOBBER)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(la), "v"(voff), "s"(rsrc) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(la), "v"(voff), "s"(rsrc) : "m0");
}
// Bytes from the first element of a tile to the end of what may be read: rows_left rows of the tensor (from the tile's
// first row on) of which cols_left columns lie at or behind the tile's first column; 0 when there is nothing.
__device__ __forceinline__ uint32_t bounded_bytes(int rows_left, int cols_left, int row_bytes) {
    const int r = rows_left < 8192 ? rows_left : 8192;      // (more than any tile has; keeps the product in 32 bits)
    return (r > 0 && cols_left > 0) ? (uint32_t)(r - 1) * (uint32_t)row_bytes + 2u * (uint32_t)cols_left : 0u;
}
static constexpr uint32_t DMA_NOTHING = 0x7ffffff0u;        // an offset beyond every bounded_bytes()

// Same for 64 x 4 bytes: lane l copies one dword to LDS address lds_uniform + 4 * l.
__device__ __forceinline__ void dma4(const void* gbase_uniform, uint32_t voff, uint32_t lds_uniform) {
    const uint32_t la = __builtin_amdgcn_readfirstlane(lds_uniform);
    const uint64_t gb = (uint64_t)(uintptr_t)gbase_uniform;
    const uint32_t glo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gb);
    const uint32_t ghi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gb >> 32));
    const uint64_t gu = (uint64_t)glo | ((uint64_t)ghi << 32);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(la), "v"(voff), "s"(gu) : "memory", "m0");
}

// a 16-bit store (low half of `data`) that the compiler's own wait counts know nothing of
__device__ __forceinline__ void store16_uncounted(const void* gbase_uniform, uint32_t voff, uint32_t data) {
    const uint64_t gb = (uint64_t)(uintptr_t)gbase_uniform;
    const uint32_t glo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)gb);
    const uint32_t ghi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(gb >> 32));
    const uint64_t gu = (uint64_t)glo | ((uint64_t)ghi << 32);
    asm volatile("s_nop 4\n\tglobal_store_short %0, %1, %2" :: "v"(voff), "v"(data), "s"(gu) : "memory");
}

// workgroup barrier without the fence a __syncthreads() carries (that fence would wait for
// every outstanding global->LDS load, i.e. drain the pipeline)
__device__ __forceinline__ void barrier_nofence() { asm volatile("s_barrier" ::: "memory"); }

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// wait until at most n (wave-uniform, 0..63) vector-memory operations of this wave are pending
__device__ __forceinline__ void wait_vmcnt_dyn(int n) {
    switch (n) {
#define TFLA_W(k) case k: wait_vmcnt<k>(); break;
        TFLA_W(0) TFLA_W(1) TFLA_W(2) TFLA_W(3) TFLA_W(4) TFLA_W(5) TFLA_W(6) TFLA_W(7) TFLA_W(8) TFLA_W(9)
        TFLA_W(10) TFLA_W(11) TFLA_W(12) TFLA_W(13) TFLA_W(14) TFLA_W(15) TFLA_W(16) TFLA_W(17) TFLA_W(18)
        TFLA_W(19) TFLA_W(20) TFLA_W(21) TFLA_W(22) TFLA_W(23) TFLA_W(24) TFLA_W(25) TFLA_W(26) TFLA_W(27)
        TFLA_W(28) TFLA_W(29) TFLA_W(30) TFLA_W(31) TFLA_W(32) TFLA_W(33) TFLA_W(34) TFLA_W(35) TFLA_W(36)
        TFLA_W(37) TFLA_W(38) TFLA_W(39) TFLA_W(40) TFLA_W(41) TFLA_W(42) TFLA_W(43) TFLA_W(44) TFLA_W(45)
        TFLA_W(46) TFLA_W(47) TFLA_W(48) TFLA_W(49) TFLA_W(50) TFLA_W(51) TFLA_W(52) TFLA_W(53) TFLA_W(54)
        TFLA_W(55) TFLA_W(56) TFLA_W(57) TFLA_W(58) TFLA_W(59) TFLA_W(60) TFLA_W(61) TFLA_W(62) TFLA_W(63)
#undef TFLA_W
        default: wait_vmcnt<0>(); break;
    }
}

// Asynchronous fill of a [ROWS][COLS] bf16 tile.  init() precomputes the per-lane byte offsets
// into the global tile (they depend only on the global row stride), issue() launches this
// wave's share of the loads: N instructions of 64 x 16 bytes.
template <int ROWS, int COLS, int NT, int KIND> struct DmaTile {
    static constexpr int CPR = COLS / 8, TOTAL = ROWS * CPR, NWV = NT / 64, N = TOTAL / (64 * NWV);
    static_assert(TOTAL % (64 * NWV) == 0 && N >= 1, "tile must split into whole wave loads");
    uint32_t goff[N];
    __device__ __forceinline__ void init(long gstride_elems, int tid) {
        const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int q = (wave + j * NWV) * 64 + lane;
            const int r = q / CPR, pc = q % CPR;
            const int c = pc ^ swz_mask<KIND, CPR>(r);
            goff[j] = (uint32_t)((r * gstride_elems + c * 8) * 2);
        }
    }
    // gtile: wave-uniform address of the tile's first element; lds: LDS address of the tile
    // ONCE: with the non-temporal hint (a tile that no other workgroup reads)
    template <bool ONCE = false>
    __device__ __forceinline__ void issue(const bf16_t* gtile, uint32_t lds, int tid) const {
        const int wave = tid >> 6;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if constexpr (ONCE) dma16_nt(gtile, goff[j], lds + (wave + j * NWV) * 1024);
            else dma16(gtile, goff[j], lds + (wave + j * NWV) * 1024);
        }
    }
    // The loads j = part, part + nparts, ... of a tile that reaches past the end of its tensor: `bytes` as
    // bounded_bytes() gives it (rows past the end lie beyond it), cols_left the columns that exist from the tile's first
    // on (the lanes behind them are sent out of range).
    template <bool CLOBBER>
    __device__ __forceinline__ void issue_bounded(const bf16_t* gtile, uint32_t bytes, int cols_left, uint32_t lds, int tid,
                                                  int part = 0, int nparts = 1) const {
        const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (j % nparts == part) {
                uint32_t vo = goff[j];
                if (cols_left < COLS) {
                    const int q = (wave + j * NWV) * 64 + lane;
                    const int c = (q % CPR) ^ swz_mask<KIND, CPR>(q / CPR);
                    vo = c * 8 < cols_left ? vo : DMA_NOTHING;
                }
                dma16_bounded<CLOBBER>(gtile, bytes, vo, lds + (wave + j * NWV) * 1024);
            }
    }
    // For tiles that all end at the same column: sends the lanes behind it out of range once; issue_bounded() is then given
    // COLS.  (Found again at every request before: 16 heads of 96 / 192, batch 2, 3000 steps, forward + backward 213 -> 207 us;
    // 8 heads of 256 / 512 within 0.5 %.)
    __device__ __forceinline__ void bound_columns(int cols_left, int tid) {
        const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int q = (wave + j * NWV) * 64 + lane;
            const int c = (q % CPR) ^ swz_mask<KIND, CPR>(q / CPR);
            goff[j] = c * 8 < cols_left ? goff[j] : DMA_NOTHING;
        }
    }
    // the loads j = part, part + nparts, ... only (part, nparts compile-time in the callers)
    template <bool ONCE = false>
    __device__ __forceinline__ void issue_part(const bf16_t* gtile, uint32_t lds, int tid, int part, int nparts) const {
        const int wave = tid >> 6;
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (j % nparts == part) {
                if constexpr (ONCE) dma16_free_nt(gtile, goff[j], lds + (wave + j * NWV) * 1024);
                else dma16_free(gtile, goff[j], lds + (wave + j * NWV) * 1024);
            }
    }
};

// Per-lane byte offsets for k-contiguous fragment reads from a SWZ_K tile with COLS columns:
// fragment (step ks, lane group g) of row (32 * blk + l32).
template <int COLS> struct KFragReader {
    static constexpr int CPR = COLS / 8, XM = CPR >= 16 ? 16 : CPR, NJ = XM / 2, RB = COLS * 2;
    uint32_t off[NJ];
    __device__ __forceinline__ void init(int l32, int g) {
        const int x = swz_mask<SWZ_K, CPR>(l32) ^ g;
#pragma unroll
        for (int j = 0; j < NJ; ++j) off[j] = (uint32_t)(l32 * RB + (((2 * j) ^ x) * 16));
    }
    // KS and BLK are compile-time in all callers (unrolled loops), so the address is off[] + constant
    __device__ __forceinline__ bf16x8 load(const char* tile, int ks, int blk) const {
        return *reinterpret_cast<const bf16x8*>(tile + off[ks % NJ] + (ks / NJ) * (XM * 16) + blk * 32 * RB);
    }
};

// Per-lane byte offsets for transposing fragment reads from a SWZ_T tile [k rows][COLS n]:
// the fragment of column block nb whose eight k values are rows
//   rowconst + ROWG * g + (lane & 15) / 4 + {0..3}  and the same + 8 * HSTEP ... (see load()).
template <int COLS> struct TFragReader {
    static constexpr int CPR = COLS / 8, NB = COLS / 32, NJ = NB < 4 ? NB : 4, RB = COLS * 2;
    uint32_t off[NJ];
    // rowg: row offset contributed by the lane group g (4 for operands chained to an MFMA
    // result, 8 for the natural k order)
    __device__ __forceinline__ void init(int lane, int rowg) {
        const int i = lane & 15, m = lane >> 4, g = lane >> 5;
        const int row = rowg * g + (i >> 2);
        const int f = swz_mask<SWZ_T, CPR>(i >> 2);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            off[j] = (uint32_t)(row * RB + (((4 * j) ^ f) + 2 * (m & 1) + ((i & 3) >> 1)) * 16 + (i & 1) * 8);
    }
    // byte offset of column block nb for this lane; for callers whose nb is not a compile-time value
    // (indexing off[] with a run-time value would push the array out of registers)
    __device__ __forceinline__ uint32_t block_offset(int nb) const {
        uint32_t o = off[0];
#pragma unroll
        for (int j = 1; j < NJ; ++j) o = (nb % NJ == j) ? off[j] : o;
        return o + (uint32_t)(nb / NJ) * 256u;
    }
    // the same for a run-time nb without the table
    static __device__ __forceinline__ uint32_t offset_of(int lane, int rowg, int nb) {
        const int i = lane & 15, m = lane >> 4, g = lane >> 5;
        const int row = rowg * g + (i >> 2), f = swz_mask<SWZ_T, CPR>(i >> 2);
        return (uint32_t)(row * RB + (((4 * (nb % NJ)) ^ f) + 2 * (m & 1) + ((i & 3) >> 1)) * 16 + (i & 1) * 8) + (uint32_t)(nb / NJ) * 256u;
    }
    // the same fragment read from a precomputed block_offset()
    static __device__ __forceinline__ bf16x8 load_at(const char* tile, uint32_t boff, int rowA, int rowB) {
        const char* p = tile + boff;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (__attribute__((address_space(3))) bf16x4*)(p + rowA * RB));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (__attribute__((address_space(3))) bf16x4*)(p + rowB * RB));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
    // rows rowA.. and rowB.. (multiples of 4, before the lane part) give elements 0..3 and 4..7
    __device__ __forceinline__ bf16x8 load(const char* tile, int nb, int rowA, int rowB) const {
        const char* p = tile + off[nb % NJ] + (nb / NJ) * 256;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (__attribute__((address_space(3))) bf16x4*)(p + rowA * RB));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (__attribute__((address_space(3))) bf16x4*)(p + rowB * RB));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
};

// Prefetch into the XCD's L2 for the recurrent kernels: the workgroups that hold the state tiles of one (batch, head) read the
// same rows of X and Y at about the same time, so all their requests together wait for one trip to memory per line, and what is
// on its way is a fraction of what the rings hold.  Here every one of them requests its share of the 128-byte lines of a piece
// AHEAD pieces ahead, four bytes per line, into a scrap of LDS that nobody reads.
template <int BK, int AHEAD> struct LinePrefetch {
    bool on = false;
    const char* base;
    uint32_t vo, dst;
    int row, sub = 0, left, rows, ld2;
    // T: one of the two tensors (rows of `ld` values, `steps` of them per (batch, head)) of whose `width` columns the
    // `sharers` workgroups read all; this one is number `index`.  P pieces, the first at row0.
    __device__ __forceinline__ void init(const void* T, long bh, int ld, int steps, int width, int sharers, int index, int P, long row0, int lane,
                                         uint32_t scrap) {
        const int lpr = width / 64, per = BK * lpr / sharers;         // lines per row, lines per workgroup
        // Whole shares of at most one line per lane.  With eight sharers (heads of 256, of 128 / 256) and on short sequences
        // there is nothing to gain: 64 heads of 256, 2048 steps 65 / 58 us per launch without, 67 / 60 with.
        // Nor with more than an XCD runs at a time (32), whose shares come too late or into other L2s: 4 sequences of 4 heads of
        // 1024, 128 sharers, 4096 steps, forward + backward 2745 us without, 2774 with.
        on = sharers >= 16 && sharers <= 32 && P >= 4 * AHEAD && per >= 1 && per <= 64 && per * sharers == BK * lpr && steps >= BK && ((uintptr_t)T & 3) == 0;
        base = reinterpret_cast<const char*>(T) + bh * steps * (long)ld * 2;
        const int q = index * per + (lane < per ? lane : per - 1);
        const int col = (q % lpr) * 128;
        vo = (uint32_t)((q / lpr) * ld * 2 + (col < ld * 2 ? col : ld * 2 - 16));
        dst = scrap; row = (int)row0; left = P - 1; rows = steps; ld2 = ld * 2;
    }
    __device__ __forceinline__ void advance(int PPC, int step_rows, int wrap_rows) {
        if (left <= 0) return;
        --left;
        const bool wrap = ++sub == PPC;
        row += wrap ? wrap_rows : step_rows;
        if (wrap) sub = 0;
    }
    // one load per call, also where the piece is not there to prefetch: callers count them
    __device__ __forceinline__ void issue() const { dma4(base + (long)(row + BK <= rows ? row : 0) * ld2, vo, dst); }
};

}  // namespace tfla
