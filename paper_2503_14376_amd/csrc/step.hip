// Single-step recurrent kernel (paper Sec. 2.1 for mLSTMexp, Sec. 4.1 for mLSTMsig): the form
// used for generation, where the state (C, n, m) is read and written once per step.  The
// step is bound by the traffic of the matrix memory C (App. F, memory operation counts of the
// recurrent formulation): 2 d_qk d_hv floats per head.
//
// One workgroup owns all d_qk rows of a slab of COLS columns of C for one (batch, head): COLS / 4 lanes side by side hold
// four columns each, the other lanes further rows, so every row segment moves as one coalesced access.  C is updated in
// registers between its load and its store (both non-temporal: the state is touched once per step), and the numerator C'^T q~ needs one reduction over the rows.  The rows are
// taken in batches of U per lane, the next batch requested before the present one is used and the first before anything
// else, so that the gates, the normaliser and the staging of q and k hide behind it.
// The normaliser n' q~ and the max state are recomputed by every slab (d_qk values).
#include "tfla_device.h"
#include "tfla_internal.h"

namespace tfla {

template <typename DT, int COLS, int U>
__global__ void __launch_bounds__(256) step_kernel(StepArgs a) {
    using E = Elem<DT>;
    constexpr int LPR = COLS / 4, RP = 256 / LPR;    // lanes per row segment, rows per pass
    __shared__ float sk[1024], sq[1024];
    __shared__ float snum[4][COLS];
    __shared__ float sred[4];
    const int bh = blockIdx.y, nb = blockIdx.x, tid = threadIdx.x, tx = tid % LPR, ty = tid / LPR;
    const int dqk = a.dqk, dhv = a.dhv;
    const bool is_exp = a.variant == 0;
    const float* Cin = a.C + ((long)bh * dqk) * dhv + nb * COLS + 4 * tx;
    float* Cout = a.C_out + ((long)bh * dqk) * dhv + nb * COLS + 4 * tx;
    f32x4 c[U];
    auto load_batch = [&](int m0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m = m0 + u * RP + ty;
            if (m < dqk) c[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(Cin + (long)m * dhv));
        }
    };
    load_batch(0);
    const DT* q = reinterpret_cast<const DT*>(a.q) + (long)bh * dqk;
    const DT* k = reinterpret_cast<const DT*>(a.k) + (long)bh * dqk;
    const DT* v = reinterpret_cast<const DT*>(a.v) + (long)bh * dhv + nb * COLS;
    float ip = a.i_pre[bh], fp = a.f_pre[bh];
    if (a.softcap > 0.0f) { ip = a.softcap * tanhf(ip / a.softcap); fp = a.softcap * tanhf(fp / a.softcap); }
    const float qscale = 1.0f / sqrtf((float)dqk);
    // gates (Sec. 2.1: m_t = max(log sigma(f~) + m_{t-1}, i~), stabilised f', i'; Sec. 4.1: sigmoids)
    float fg, ig, m_new = 0.0f;
    if (is_exp) {
        const float fbar = fminf(fp, 0.0f) - log1pf(expf(-fabsf(fp)));
        const float m_old = a.m ? a.m[bh] : 0.0f;
        m_new = fmaxf(fbar + m_old, ip);
        fg = expf(fbar + m_old - m_new);
        ig = expf(ip - m_new);
    } else {
        fg = 1.0f / (1.0f + expf(-fp));
        ig = 1.0f / (1.0f + expf(-ip));
    }
    for (int i = tid; i < dqk; i += 256) {
        sk[i] = E::to_f32(k[i]);
        sq[i] = E::to_f32(q[i]) * qscale;
    }
    // normaliser: n' = f' n + i' k, dot = n'^T q~ (every slab recomputes it; slab 0 stores n').  A thread reads back
    // only what it staged itself.
    if (is_exp) {
        float dot = 0.0f;
        for (int i = tid; i < dqk; i += 256) {
            const float nn = fg * (a.n ? a.n[(long)bh * dqk + i] : 0.0f) + ig * sk[i];
            if (nb == 0 && a.n_out) a.n_out[(long)bh * dqk + i] = nn;
            dot += nn * sq[i];
        }
        dot = wave_sum(dot);
        if ((tid & 63) == 0) sred[tid >> 6] = dot;
    } else if (nb == 0) {
        // mLSTMsig has neither: zeros where the caller wants them
        if (a.n_out)
            for (int i = tid; i < dqk; i += 256) a.n_out[(long)bh * dqk + i] = 0.0f;
        if (a.m_out && tid == 0) a.m_out[bh] = 0.0f;
    }
    const f32x4 vv = {E::to_f32(v[4 * tx]), E::to_f32(v[4 * tx + 1]), E::to_f32(v[4 * tx + 2]), E::to_f32(v[4 * tx + 3])};
    __syncthreads();
    // matrix memory: C' = f' C + i' k v^T, numerator C'^T q~
    f32x4 num = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int m0 = 0; m0 < dqk; m0 += RP * U) {
        f32x4 p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) p[u] = c[u];
        load_batch(m0 + RP * U);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m = m0 + u * RP + ty;
            if (m < dqk) {
                const float ik = ig * sk[m], qm = sq[m];
                f32x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) { o[e] = fg * p[u][e] + ik * vv[e]; num[e] += o[e] * qm; }
                __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>(Cout + (long)m * dhv));
            }
        }
    }
    // over the rows of the wavefront (lanes LPR apart), then over the four wavefronts
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) num[e] += __shfl_xor(num[e], o, 64);
    if ((tid & 63) < LPR) *reinterpret_cast<f32x4*>(&snum[tid >> 6][4 * tx]) = num;
    __syncthreads();
    if (tid < COLS) {
        const float s = (snum[0][tid] + snum[1][tid]) + (snum[2][tid] + snum[3][tid]);
        float den = 1.0f;
        if (is_exp) {
            const float d = sred[0] + sred[1] + sred[2] + sred[3];
            den = fmaxf(fabsf(d), expf(-m_new)) + a.eps;
        }
        reinterpret_cast<DT*>(a.h)[(long)bh * dhv + nb * COLS + tid] = E::from_f32(s / den);
    }
    if (is_exp && nb == 0 && tid == 0 && a.m_out) a.m_out[bh] = m_new;
}

// Slabs of 64 columns for a large state (2^24 values and more over all heads: 16 sequences of 8 heads 256 / 512), of 32
// below, where the launch would otherwise leave CUs without work.  A batch covers all rows up to 256, so that a workgroup
// has its whole slab (or 256 rows of it) in flight at once; more batches of fewer rows lose 5 to 40 %.  32 / 64 columns, us
// per step: 1 sequence of 8 heads 256 / 512 5.2 / 6.4, 8 sequences 13.6 / 14.4, 32 sequences 56.5 / 55.6, 64 sequences 111 /
// 104; 4 heads of 1024, 1 sequence 13.1 / 17.3, 16 sequences 117 / 109.
// Loads and stores are non-temporal because a model of several layers comes back to a layer's state only after those of all
// the others.  us per step (replayed graph), the former kernel of plain accesses and no requests ahead / this one, states
// taken in turn from 1.6 GB: 1, 8, 16, 32, 64 sequences of 8 heads 256 / 512 12.3 / 5.2, 20.7 / 13.6, 32.2 / 28.2, 61.8 /
// 54.7 (4.9 TB/s; a large copy moves 5.0), 117 / 102.5; 16 sequences of 8 heads 512 / 512 59.3 / 55.0.  One state updated in
// place over and over, which the 256 MB memory-side cache could hold: 6.1 / 5.3, 12.5 / 10.8, 22.9 / 25.1, 43.2 / 51.7, 94.8 /
// 99.1; 43.2 / 52.5.  Plain accesses here: 41 to 45 in the last case, but 60.3 to 61.3 where the states take turns.
template <typename DT, int COLS> static void launch_step_c(const StepArgs& a, int BH, hipStream_t s) {
    const dim3 grid(a.dhv / COLS, BH), block(256);
    constexpr int U64 = COLS / 16;              // passes that cover 64 rows
    if (a.dqk <= 64) hipLaunchKernelGGL((step_kernel<DT, COLS, U64>), grid, block, 0, s, a);
    else if (a.dqk <= 128) hipLaunchKernelGGL((step_kernel<DT, COLS, 2 * U64>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((step_kernel<DT, COLS, 4 * U64>), grid, block, 0, s, a);
}
template <typename DT> static hipError_t launch_step_t(const StepArgs& a, int BH, hipStream_t s) {
    if ((long)BH * a.dqk * a.dhv >= 1L << 24) launch_step_c<DT, 64>(a, BH, s);
    else launch_step_c<DT, 32>(a, BH, s);
    return hipGetLastError();
}

hipError_t launch_step(const StepArgs& a, int BH, hipStream_t s) {
    return a.dtype == 1 ? launch_step_t<bf16_t>(a, BH, s) : launch_step_t<float>(a, BH, s);
}

}  // namespace tfla
