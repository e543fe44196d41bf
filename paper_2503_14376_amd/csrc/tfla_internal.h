// Host-side declarations shared by the translation units of libtfla_mlstm: argument blocks
// of the kernel families and their launchers.  Nothing here is exported.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace tfla {

struct FillList { float* p[4]; long n[4]; };     // arrays to zero; n[q] = 0: slot unused

// ---- chunkwise gates (App. B.2 "Chunkwise Gates", App. B.2 inter-chunk max state) ----------
struct GateArgs {
    const float* i_pre;   // (BH, Tvalid)
    const float* f_pre;   // (BH, Tvalid)
    const float* m0;      // (BH) or NULL
    int T, L, Nc, variant;
    int Tvalid;           // the caller's sequence length; steps Tvalid .. T - 1 get forget gate 1, input gate 0
    float qscale;         // 1/sqrt(dqk)
    float softcap;        // c of the gate soft-cap c tanh(x / c) on both pre-activations; 0 = none
    // outputs, all (BH, T) unless noted
    float* wrow;          // log2-domain row term of the intra-chunk weight (includes log2 qscale)
    float* ucol;          // log2-domain column term (i-bar_j - b_j) * log2(e)
    float* sH;            // inter-chunk row scale b-bar_i * qscale
    float* aK;            // a-bar_j = exp(a_j - m_k)
    float* gbar;          // (BH, Nc) g-bar_k
    float* mout;          // combined max state m_t of every step
    float* mout_user;     // (BH, Tvalid) a second copy in the caller's layout, or NULL
    float* mfinal;        // (BH) m after the last chunk, or NULL
    float* tmp;           // (BH, 3, T) scratch (values of the pre-pass's arithmetic type: doubles when `precise`)
    // fp32 kernels: pre-pass in double, and the rounding remainders of the two exponents (wrow + wrow_lo and
    // ucol + ucol_lo are the exponents to double accuracy); csum then holds doubles as well.  NULL / 0 otherwise.
    float* wrow_lo; float* ucol_lo; int precise;
    float* csum;          // (BH, 2, Nc) scratch: per-chunk sum of f-bar and max of a
    // the outputs that mLSTMsig does not have, zeroed on the way (a launch of its own for them took 5 us)
    FillList zero;
};
hipError_t launch_gates(const GateArgs& a, int BH, hipStream_t s);

// the pre-pass is one workgroup per (batch, head) instead of two launches (gates.hip has both sides)
constexpr int GATE_FUSED_CHUNKS = 16;
inline bool gates_in_one_launch(int Nc, int L) { return Nc <= GATE_FUSED_CHUNKS && (L == 64 || L == 128 || L == 256 || L == 512); }
struct GateBwdPrepArgs {
    const float* wrow; const float* sH; const float* n_out; const float* m_out;
    float* wrowB; float* sQ;
    long n; int variant; float eps;
    const float* wrow_lo; float* wrowB_lo;   // fp32 kernels: remainders of wrow / wrowB, or NULL
    int T, Tvalid;        // n_out, m_out are (BH, Tvalid), everything else (BH, T); the steps in between get den = 1
};
hipError_t launch_gate_bwd_prep(const GateBwdPrepArgs& a, hipStream_t s);

struct GateGradArgs {
    const float* partQ; int nbQ;   // (nbQ, BH*T) partial q.dq
    const float* partK; int nbK;   // (nbK, BH*T) partial k.dk
    const double* cdot;            // (BH, STATE_DOT_PARTS) partial sums of <C_T, dC_T>, or NULL
    const float* i_pre; const float* f_pre;
    float* d_i; float* d_f;
    double* bsum;                  // (BH, ceil(T / 1024)) scratch: block sums
    int T, variant; long BHT;
    int Tvalid;                    // i_pre, f_pre, d_i, d_f are (BH, Tvalid)
    float softcap;                 // as in GateArgs: the gradients are taken through the cap
    // optional anchors of the reverse cumulative sum, one per block of G chunks (G * L <= ANCHOR_STEPS): its exact value
    // just after the last step of the block, <C, dC> at that boundary, as npart partial sums per boundary
    // (RecArgs::anc_part: (BH, nslot, npart)); NULL = one scan over the whole sequence
    const float* anchor; int L, Nc, G, npart;
};
hipError_t launch_gate_grads(const GateGradArgs& a, int BH, hipStream_t s);

hipError_t launch_zero(const FillList& f, hipStream_t s);
hipError_t launch_copy(const float* from, float* to, int n, hipStream_t s);
// out[bh] = <A[bh], Bm[bh]>; A (BH, *, lda), Bm (BH, d1, d2): the first d2 columns of the first d1 rows of A's `perA` values
// as STATE_DOT_PARTS partial sums each
constexpr int STATE_DOT_PARTS = 16;
hipError_t launch_state_dot(const float* A, long perA, int lda, const float* Bm, int d1, int d2, double* out, int BH, hipStream_t s);
// Chunks per block of the anchored forget-gate gradient scan: four (a block then has at most 2048 steps, or one chunk); two for
// heads wider than 512, whatever the chunk (at most 4096 steps), where a row's dot products run over so many terms that the
// noise of a few chunks already shows (behind a norm layer the forget-gate gradient is what survives of an almost complete
// cancellation).  The workspaces are laid out by it.
constexpr int ANCHOR_STEPS = 4096;
inline int anchor_chunks(int L, int dwide) {
    if (dwide > 512) return 2;
    return 4 * L <= 2048 ? 4 : (2048 / L > 0 ? 2048 / L : 1);
}

// ---- single recurrent step (Sec. 2.1, Sec. 4.1) ------------------------------------------------
struct StepArgs {
    const void* q; const void* k; const void* v;   // (BH, dqk), (BH, dqk), (BH, dhv)
    const float* i_pre; const float* f_pre;        // (BH)
    const float* C; const float* n; const float* m;   // state before the step; n, m may be NULL (zero)
    float* C_out; float* n_out; float* m_out;      // state after the step; n_out, m_out may be NULL
    void* h;                                       // (BH, dhv)
    int dqk, dhv, variant, dtype;
    float eps;
    float softcap;                                 // gate soft-cap, 0 = none
};
hipError_t launch_step(const StepArgs& a, int BH, hipStream_t s);

// ---- NORM + output gate around the cell (Sec. 2.1 output equation; Sec. 4.1 RMS norm), transfer gains ----
struct NormArgs {
    const void* h;        // (rows, d) cell output h~, element type per dtype
    const void* o_pre;    // (rows, d) output gate pre-activations, or NULL (gate = 1)
    const float* gamma;   // (NH, d) or NULL (1)
    const float* beta;    // (NH, d) or NULL (0); LayerNorm only
    void* y;              // (rows, d)
    long rows;            // B * NH * T, row = (b * NH + head) * T + t
    int NH, T, d, kind, dtype;   // kind 0 = RMS norm, 1 = LayerNorm
    float eps;
};
hipError_t launch_norm_gate_fwd(const NormArgs& a, hipStream_t s);
struct NormBwdArgs {
    const void* h; const void* o_pre; const float* gamma; const float* beta;
    const void* dy;       // (rows, d)
    void* dh;             // (rows, d)
    void* do_pre;         // (rows, d) or NULL
    float* part;          // (BH, row blocks, 2, d) partial sums for d gamma / d beta, or NULL
    int NH, T, d, kind, dtype;
    float eps;
};
hipError_t launch_norm_gate_bwd(const NormBwdArgs& a, int BH, hipStream_t s);
int norm_row_blocks(int T);
struct NormParamGradArgs {
    const float* part; float* dgamma; float* dbeta;   // outputs (NH, d), either may be NULL
    int B, NH, nblk, d;
    int kind;                                         // 0 = RMS norm: dbeta is zero
};
hipError_t launch_norm_param_grad(const NormParamGradArgs& a, hipStream_t s);
struct GainArgs {
    const void* h; const void* v;   // (BH, T, d)
    float* g_before; float* g_after;   // (BH)
    int T, d, kind, dtype;
    float eps;
};
hipError_t launch_transfer_gain(const GainArgs& a, int BH, hipStream_t s);

// ---- inter-chunk recurrence (App. B.2 "Inter-chunk Recurrent Contribution"; App. B.3) -------
// state <- gbar[k] * state + (rs (.) X_k)^T Y_k, chunk by chunk; the state *before* each
// update is written to slot k.
struct RecArgs {
    const void* X;        // (BH, T_in, d1_in)
    const void* Y;        // (BH, T_in, d2_in)
    const float* rs;      // (BH, T)
    const float* gbar;    // (BH, Nc)
    const float* S0;      // (BH, d1_in, d2_in) fp32 or NULL (zero)
    void* stT;            // (BH, Nc, d2, d1) element type DT, or NULL
    float* Sfinal;        // (BH, d1_in, d2_in) fp32 or NULL
    float* Sfinal2;       // second copy of the final state, (BH, d1, d2), or NULL
    const float* n0;      // (BH, d1_in) or NULL; normaliser vector, forward mLSTMexp only
    float* nst;           // (BH, Nc, d1) or NULL (NULL = no normaliser vector); the bf16 kernel stores the same
                          // bytes as (BH, Nc, 2, d1) bf16: n rounded to bf16, and the rounding remainder
    float* nfinal;        // (BH, d1_in) or NULL
    int T, L, Nc, d1, d2, reverse;
    // the caller's sequence length and head dimensions: the kernels work on whole chunks and on their own widths
    // (T >= T_in, d1 >= d1_in, d2 >= d2_in) and take the steps and columns in between as zeros
    int T_in, d1_in, d2_in;
    bool padded() const { return T_in != T || d1_in != d1 || d2_in != d2; }
    // bf16 kernel only, for the anchors of the forget-gate gradient scan (the boundaries between its blocks of anc_G
    // chunks; slot s = the boundary between chunks s * anc_G - 1 and s * anc_G, slot 0 unused):
    //   anc      (forward launch) receives fp32 copies of the state at those boundaries, (BH, nslot, d1 * d2) in the
    //            order of the kernel's accumulator registers;
    //   anc_in   (reversed launch) = what the forward launch left in anc: every wavefront multiplies its part of it
    //            with its fp32 accumulators (the same element order) and leaves the partial inner product in
    //   anc_part (BH, nslot, npart), npart = (d1 / 64) * (d2 / 32) = rec_anchor_parts().
    // NULL = none.
    float* anc; const float* anc_in; float* anc_part; int anc_G;
};
hipError_t launch_recurrent(const RecArgs& a, int BH, int dtype, hipStream_t s);
// dQ and dK weight the same matrix dH V^T.  Where the contraction that forms it (over d_hv) is wider than this, the dQ
// kernel stores its weighted tiles E (L x L per chunk) and the dK kernel reads them; up to this width both kernels
// form the matrix themselves, because E is then more bytes than the operands it replaces (measured at
// d_hv = 64 / 128 / 256: -19 % / -8 % / -1 % per step without E; at 512: +3 %).
#ifndef TFLA_NOE_MAX_D1
#define TFLA_NOE_MAX_D1 256
#endif
inline bool tile_shares_E(int dhv) { return dhv > TFLA_NOE_MAX_D1; }

inline int rec_anchor_parts(int d1, int d2) { return (d1 / 64) * (d2 / 32); }

// ---- intra-chunk tiled kernels (Sec. 3, App. C.3 Alg. 1, App. C.4) ---------------------------
// out[r,:] = sum_c exp2(wrow[r] + wcol[c]) * (X_r . Y_c) * Z_c  (causal within the chunk)
//            + srow[r] * (X_r St)
enum { MODE_H = 0, MODE_DV = 1, MODE_DQ = 2, MODE_DK = 3 };
struct TileArgs {
    const void* X; const void* Y;   // (BH, out_T, in_ld1)
    const void* Z; void* Out;       // (BH, out_T, out_ld), see below
    const float* wrow; const float* wcol; const float* srow;   // (BH, T)
    const void* St;                 // (BH, Nc, d_hv, d_qk): d2 x d1 for H and dV, d1 x d2 for dQ and dK
    int T, L, Nc, d1, d2;
    int kc_desc;                    // bf16 kernels: walk the chunks last to first (set by the launcher)
    // MODE_H, mLSTMexp: normaliser
    int variant; float eps;
    const float* nstate;            // (BH, Nc, d1); bf16 kernels: (BH, Nc, 2, d1) bf16 as RecArgs::nst
    const float* mout;              // (BH, T)
    float* nout;                    // (BH, out_T) or NULL
    // MODE_H, mLSTMexp: the backward pass's row weights with 1 / h_denom folded in (what gate_bwd_prep_kernel
    // computes from n_out and m_out), written here while the denominator is at hand; (BH, T) each, or NULL
    float* wrowB_out; float* sQ_out;
    // MODE_DQ / MODE_DK: partial row dots  sum_n out[r,n] * dotwith[r,n]
    const void* dotwith;            // (BH, out_T, out_ld)
    float* dotpart;                 // (d2/BD2, BH*T)
    // bf16 MODE_DQ writes, bf16 MODE_DK reads: the weighted matrix E of every chunk, (BH, Nc, L, L)
    void* E;
    // Contractions wider than the kernels hold in registers.  bf16, above 512: a launch before the mode's own leaves the weighted
    // matrix in memory (tile_weights.h), dQ's in E, the others' in part_acc, for H with the sums of its rows behind it.  fp32, above
    // 256, and H of bf16 where that does not fit (weights_fit()): every term of the result is linear in the products over d1, so the
    // launcher runs the kernel once per half and the halves meet in fp32.  The caller provides the buffers; the remaining fields
    // are filled in by the launcher.
    float* part_acc;                // (BH, T, d2) unnormalised result of the first half; or (BH, Nc, L, L) weights, bf16
    float* part_nrm;                // (BH, T) its share of the normaliser (MODE_H, mLSTMexp)
    const float* acc_in; const float* nrm_in;   // add these to the accumulators / normaliser before the epilogue
    float* acc_out; float* nrm_out;             // store the raw accumulators / normaliser instead of the output
    // The caller's tensors are read and written where they are also when the sequence ends inside its last chunk or a
    // head dimension lies between the kernels' widths: their first d1-wide operands have in_ld1 columns (in_cols1 of
    // them behind the pointer: less than in_ld1 in the second half of a split contraction), their d2-wide ones out_ld,
    // and all of them out_T steps; everything past that is taken as zero and not stored.  Nothing is padded:
    // out_T = T, in_ld1 = in_cols1 = the contraction's whole width, out_ld = d2.  All are multiples of 8 (out_T is not).
    int out_T, out_ld, in_ld1, in_cols1;
    // fp32 kernels: rounding remainders of the row and column exponents (the weight is exp2 of the sum of all four),
    // and where MODE_H leaves the remainder that belongs to wrowB_out; NULL = none
    const float* wrow_lo; const float* wcol_lo; float* wrowB_lo_out;
    // bf16 kernels, filled in by the launcher: what the decomposition of the linear workgroup id divides by --
    // batch*head count, slices per XCD, and for each divisor its log2 when it is a power of two, else -1
    // (a division by a run-time value costs the start of every workgroup some forty instructions)
    int dec_bh, dec_bpx, sh_gx, sh_gy, sh_bpx, sh_nc;
    // bf16 MODE_H, fused layer output (Sec. 2.1, hidden-state output equation: y = sigma(o~) (.) NORM(h~)), where one
    // workgroup holds whole rows of h~ (d2 equal to the width of its column block, nothing padded): fz_y != NULL makes
    // the kernel store y (BH, T, d2) next to h~.  fz_o: (BH, T, d2) gate pre-activations or NULL (gate = 1);
    // fz_gamma / fz_beta: (fz_NH, d2) or NULL; fz_kind 0 = RMS norm, 1 = LayerNorm (as NormArgs).
    const void* fz_o; const float* fz_gamma; const float* fz_beta; void* fz_y;
    int fz_kind, fz_NH; float fz_eps;
};
// what the layer's forward entry point hands down to the H kernel when the fusion applies
struct LayerFuse {
    const void* o_pre; const float* gamma; const float* beta; void* y;
    int kind, NH; float eps;
};
template <int MODE> hipError_t launch_tile_mode(const TileArgs& a, int BH, int dtype, hipStream_t s);
// d2 block of a tiled kernel (mode MODE_*) with contraction width d1; rows = batch*head x steps.
// 128 columns keep a bf16 wavefront within 256 registers, so that two workgroups share a CU when d1 <= 256.  From
// d1 = 512 on a workgroup's own X rows fill half of the register file and one workgroup takes the CU in any case: a
// 256-wide block then halves how often the X rows and the column tiles are fetched and the score tile is computed (forward
// + backward, 8 heads of 512, batch 4, 4096 steps: 1.418 -> 1.335 ms); at d1 = 1024 it halves how often the X rows and the
// weights in memory are fetched.  It pays only while its workgroups still cover the 256 CUs: at 64
// workgroups (8 heads of 512, 512 steps, forward) it measured 40.5 us against 36.0 us for 128 columns, at 128
// workgroups (1024 steps, forward + backward) 155 against 144 us.
// (The 256-wide instantiations exist for the four-wavefront workgroups only, i.e. for chunk sizes that are
// multiples of 128.)
// tile_width_override (set through tfla_tile_width, a measurement aid for tile-size sweeps): 0 = the choice
// described above; 64 / 128 force that width wherever it divides d2; 256 changes nothing (it is already taken
// wherever it is built).  The workspace layout depends on the width, so it must not change between the
// workspace query, the forward call and the backward call of one step.
// A contraction over 1024 columns (bf16): whether the weighted matrix of H, L values per row, and the sums of its rows, one per 64
// columns at most, fit where the fp32 partial results of a split contraction would lie: d_hv values per row, a size that callers
// have planned with.  (The other modes have memory that is sized for the matrix.)
inline bool weights_fit(int L, int d2, int mode) { return mode != MODE_H || 2 * L + L / 16 <= 4 * d2; }
extern int tile_width_override;
inline int tile_bd2(int d1, int d2, int dtype, int L, long rows) {
    const int ov = tile_width_override;
    if (dtype == 1 && (ov == 64 || ov == 128) && d2 % ov == 0) return ov;
    if (dtype == 1 && d1 >= 512 && d2 % 256 == 0 && L % 128 == 0 && (rows / 128) * (d2 / 256) >= 256) return 256;
    // fp32: 64 columns while 128 would leave fewer than 512 workgroups of two wavefronts
    if (d2 % 128 == 0 && (dtype == 1 || (rows / 64) * (d2 / 128) >= 512)) return 128;
    return 64;
}
// dV, dQ and dK in one launch (tile_grads.hip), where dQ and dK need not hand E over.
// bf16: d_hv up to 256, and every part fits two workgroups per CU (contractions up to 256 columns; wider ones hold their X rows
// in half of the register file), with the block widths that kernel is built for (tile_width_override may ask for others).
// Faster at every size measured, 6 to 37 % of forward + backward, from one sequence of 777 steps to 128 heads of 32.
// fp32: the same widths.  What the kernels wait for there is the matrix unit, and what one launch gains is the chip filled
// once instead of three times: 44 % of forward + backward for one head of 64 and 256 steps, 24 % for 8 heads of 256 and 500
// steps, 2 to 12 % where each launch fills it many times over.  In the middle, two-wavefront workgroups (chunk sizes that are
// no multiple of 128) of a 256-wide d_hv and a narrow d_qk: from 32768 rows on the three launches have 128-wide blocks for a
// d_qk of 128 as well (tile_bd2), and how full each launch's last round of workgroups is decides.  us, three launches / one:
// 128 / 256, 24576 rows 353 / 298, 32768 rows 317 / 337, 49152 rows 523 / 514, chunk 192 and 36864 rows 521 / 470; 64 / 256, 32768 rows
// 228 / 242, 49152 rows 356 / 348, 57344 rows 395 / 404.  They keep the three there; wide heads do from 65536 rows on.
inline bool grads_in_one_launch(int dqk, int dhv, int dtype, int L, long rows) {
    if (dqk > 256 || dhv > 256) return false;
    if (dtype != 1) return (dqk <= 128 && dhv <= 128) || rows < (L % 128 != 0 && dhv > 128 && dqk <= 128 ? 32768 : 65536);
    return tile_bd2(dqk, dhv, dtype, L, rows) == (dhv >= 128 ? 128 : 64) && tile_bd2(dhv, dqk, dtype, L, rows) == (dqk >= 128 ? 128 : 64);
}
// fp32, all three in one launch: 64-column blocks while 128 would leave fewer than 512 workgroups of two wavefronts (never
// narrower than tile_bd2(), whose launches have the chip to themselves: 16 heads of 128 / 256, 1024 steps 128 wide)
inline bool grads_f32_wide(int dqk, int dhv, long rows) { return (rows / 64) * (dhv / 128 + 2 * (dqk / 128)) >= 512; }
// (defined for DQK = 64, 128 and 256, each in a unit of its own that holds that width's kernels)
template <int DQK> hipError_t launch_tile_grads(const TileArgs& dv, const TileArgs& dq, const TileArgs& dk, int BH, int dtype, hipStream_t s);
// the fused layer output needs whole rows of h~ in one workgroup of the H kernel
inline bool layer_fusion_applies(int dqk, int dhv, int dtype, int L, long rows) {
    return dtype == 1 && dqk <= 512 && (dhv == 64 || dhv == 128) && tile_bd2(dqk, dhv, dtype, L, rows) == dhv;
}

}  // namespace tfla
