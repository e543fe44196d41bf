// Gate kernels: chunkwise log gates and max states (forward and backward preparation) and
// the final gate-gradient reduction.  All scalar-per-step work of the method lives here;
// it is VALU + wavefront-scan work on (B*NH*T) floats.
#include <type_traits>

#include "tfla_device.h"
#include "tfla_internal.h"

namespace tfla {

static constexpr float LOG2E = 1.4426950408889634f;

__device__ __forceinline__ float log_sigmoid(float x) { return fminf(x, 0.0f) - log1pf(expf(-fabsf(x))); }
// gate soft-cap c tanh(x / c) (App. E, soft-capping equation); c = 0 leaves x as it is
__device__ __forceinline__ float soft_cap(float x, float c) { return c > 0.0f ? c * tanhf(x / c) : x; }
__device__ __forceinline__ float soft_cap_grad(float x, float c) {
    if (!(c > 0.0f)) return 1.0f;
    const float t = tanhf(x / c);
    return 1.0f - t * t;
}
__device__ __forceinline__ float sigmoid_neg(float x) {  // sigma(-x), no overflow
    const float e = expf(-fabsf(x));
    return x >= 0.0f ? e / (1.0f + e) : 1.0f / (1.0f + e);
}

// The pre-pass is written over an arithmetic type AT.  float serves the bf16 kernels.  The fp32 kernels get the
// pre-pass in double (AT = double) and its two exponents as a (rounded, remainder) pair of floats each: the row and the
// column term of a weight both have the size of the chunk's cumulative log forget gate and nearly cancel, so a single
// float per term limits a weight to the fp32 spacing at that size (2.4e-4 at |sum f-bar| = 2560), while the sum of two
// such pairs is exact to fp32 again.
template <typename AT> __device__ __forceinline__ AT log_sigmoid_t(AT x);
template <> __device__ __forceinline__ float log_sigmoid_t<float>(float x) { return log_sigmoid(x); }
template <> __device__ __forceinline__ double log_sigmoid_t<double>(double x) { return fmin(x, 0.0) - log1p(exp(-fabs(x))); }
template <typename AT> __device__ __forceinline__ AT soft_cap_t(AT x, float c);
template <> __device__ __forceinline__ float soft_cap_t<float>(float x, float c) { return soft_cap(x, c); }
template <> __device__ __forceinline__ double soft_cap_t<double>(double x, float c) { return c > 0.0f ? (double)c * tanh(x / (double)c) : x; }
template <typename AT> __device__ __forceinline__ AT max_t(AT x, AT y);
template <> __device__ __forceinline__ float max_t<float>(float x, float y) { return fmaxf(x, y); }
template <> __device__ __forceinline__ double max_t<double>(double x, double y) { return fmax(x, y); }
template <typename AT> __device__ __forceinline__ AT exp_t(AT x);
template <> __device__ __forceinline__ float exp_t<float>(float x) { return expf(x); }
template <> __device__ __forceinline__ double exp_t<double>(double x) { return exp(x); }

// this thread's share of the arrays to zero, of `threads` in the launch
__device__ __forceinline__ void zero_share(const FillList& f, long thread, long threads) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
        for (long i = thread; i < f.n[q]; i += threads) f.p[q][i] = 0.0f;
}

// Scans over the wavefront: within the rows of 16 lanes by moves between lanes (DPP row shifts), across the four rows by
// the rows' totals, read into scalar registers.  (A shuffle through LDS per step, six per scan and as many for a sum: us per
// launch, shuffles / this, 8 heads of 8 chunks of 128 6.1 / 5.3; in double, 1 head of 4 chunks of 64 4.1 / 3.1.)
// x of the lane CTRL says, `none` where there is no such lane in the row
template <int CTRL, typename T> __device__ __forceinline__ T row_move(T x, T none) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, none), __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
    } else {
        typedef int i2 __attribute__((ext_vector_type(2)));
        const i2 n = __builtin_bit_cast(i2, none), v = __builtin_bit_cast(i2, x);
        const i2 r = {__builtin_amdgcn_update_dpp(n[0], v[0], CTRL, 0xf, 0xf, false), __builtin_amdgcn_update_dpp(n[1], v[1], CTRL, 0xf, 0xf, false)};
        return __builtin_bit_cast(T, r);
    }
}
template <typename T> __device__ __forceinline__ T lane_value(T x, int l) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
    } else {
        typedef int i2 __attribute__((ext_vector_type(2)));
        const i2 v = __builtin_bit_cast(i2, x);
        const i2 r = {__builtin_amdgcn_readlane(v[0], l), __builtin_amdgcn_readlane(v[1], l)};
        return __builtin_bit_cast(T, r);
    }
}
// the operands of op are in lane order: op(earlier lanes, later lanes)
template <typename T, typename Op> __device__ __forceinline__ T wave_excl_scan(T x, T none, int lane, Op op, T* total = nullptr) {
    x = op(row_move<0x111>(x, none), x);        // row_shr:1, 2, 4, 8
    x = op(row_move<0x112>(x, none), x);
    x = op(row_move<0x114>(x, none), x);
    x = op(row_move<0x118>(x, none), x);
    const T t0 = lane_value(x, 15), t1 = op(t0, lane_value(x, 31)), t2 = op(t1, lane_value(x, 47));
    if (total) *total = op(t2, lane_value(x, 63));
    const T before = lane < 16 ? none : lane < 32 ? t0 : lane < 48 ? t1 : t2;
    return op(before, row_move<0x111>(x, none));
}
// the same over the lanes behind
template <typename T, typename Op> __device__ __forceinline__ T wave_excl_rscan(T x, T none, int lane, Op op) {
    x = op(x, row_move<0x101>(x, none));        // row_shl:1, 2, 4, 8
    x = op(x, row_move<0x102>(x, none));
    x = op(x, row_move<0x104>(x, none));
    x = op(x, row_move<0x108>(x, none));
    const T t3 = lane_value(x, 48), t2 = op(lane_value(x, 32), t3), t1 = op(lane_value(x, 16), t2);
    const T after = lane >= 48 ? none : lane >= 32 ? t3 : lane >= 16 ? t2 : t1;
    return op(row_move<0x101>(x, none), after);
}
template <typename AT> __device__ __forceinline__ AT wave_excl_scan_add(AT v, int lane, AT* total = nullptr) {
    return wave_excl_scan(v, (AT)0, lane, [](AT x, AT y) { return x + y; }, total);
}
template <typename AT> __device__ __forceinline__ AT wave_excl_rscan_add(AT v, int lane) {
    return wave_excl_rscan(v, (AT)0, lane, [](AT x, AT y) { return x + y; });
}
template <typename AT> __device__ __forceinline__ AT wave_excl_scan_max(AT v, int lane) {
    return wave_excl_scan(v, (AT)-INFINITY, lane, [](AT x, AT y) { return max_t<AT>(x, y); });
}
// (every lane gets the result)
template <typename T, typename Op> __device__ __forceinline__ T wave_reduce(T x, Op op) {
    x = op(x, row_move<0x128>(x, x));           // row_ror:8, 4, 2, 1
    x = op(x, row_move<0x124>(x, x));
    x = op(x, row_move<0x122>(x, x));
    x = op(x, row_move<0x121>(x, x));
    return op(op(lane_value(x, 0), lane_value(x, 16)), op(lane_value(x, 32), lane_value(x, 48)));
}
template <typename AT> __device__ __forceinline__ AT wave_sum_t(AT x) { return wave_reduce(x, [](AT p, AT q) { return p + q; }); }
template <typename AT> __device__ __forceinline__ AT wave_max_t(AT x) { return wave_reduce(x, [](AT p, AT q) { return max_t<AT>(p, q); }); }

// The gate pre-pass runs as two kernels, each with one wavefront per chunk (four chunks per
// workgroup), so that it fills the chip also when batch * heads is small.
//
// Kernel 1, for chunk k: b = cumsum(f-bar), a = reverse cumsum shifted by one + i-bar (the stable
// form of App. B.2), the running maximum of (i-bar_j - b_j), and the chunk summaries g_k = sum
// f-bar and max_j a_j.
// Kernel 2: every workgroup first runs the scalar recurrence m_k = max(g_k + m_{k-1}, max_j a_kj)
// over all chunks of its (batch, head) -- as a scan: the maps m -> max(m + g, c) compose to
// (g1 + g2, max(c1 + g2, c2)) -- and then forms the per-step quantities the matrix kernels
// consume for its own chunks.
//
// The intra-chunk row maximum is separable: max_{j<=i}(b_i - b_j + i-bar_j) = b_i +
// cummax_j(i-bar_j - b_j), so the combined max state m_i = b_i + max(m_{k-1}, cummax_i) is known
// before any matrix product and no online rescaling is needed in the tiled kernel.
static constexpr int GATE_WAVES = 4;

// E consecutive values of a lane, one vector access.  What bounds these kernels is latency: few wavefronts, each with chains
// of scans, logarithms and exponentials between its loads and stores, so the accesses are few and the loads come first.  us per
// launch, value by value / as vectors, chunk and step kernel: 8 heads of 32 chunks of 256 8.6 / 6.8 and 5.4 / 4.9; 8 heads of 64 chunks
// of 512 13.5 / 10.4 and 11.6 / 6.4; the anchored gradients, 8 heads of 8192 steps 8.6 / 6.6.
template <int E, typename T> __device__ __forceinline__ void load_steps(T (&v)[E], const T* p) {
    typedef T vec __attribute__((ext_vector_type(E)));
    const vec w = *reinterpret_cast<const vec*>(p);
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = w[e];
}
// ALIGN: what p is a multiple of, where that may be less than the vector's size (the caller's tensors)
template <int E, int ALIGN = 0, typename T> __device__ __forceinline__ void store_steps(T* p, const T (&v)[E]) {
    typedef T vec __attribute__((ext_vector_type(E), aligned(ALIGN > 0 ? ALIGN : E * sizeof(T))));
    vec w;
#pragma unroll
    for (int e = 0; e < E; ++e) w[e] = v[e];
    *reinterpret_cast<vec*>(p) = w;
}

// WHOLE: a lane has exactly EC steps (chunks of 64, 128, 256 and 512), which move as vectors.
// EC > 0: the lane's E <= EC steps keep their log gates in registers (one evaluation of the logarithms per
// step instead of one per pass); EC = 0: any E, the log gates are evaluated again in every pass.
// tmp and csum hold values of type AT.
template <int EC, typename AT, bool WHOLE>
__global__ void __launch_bounds__(GATE_WAVES * 64) gates_chunk_kernel(GateArgs a) {
    const int bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kc = blockIdx.x * GATE_WAVES + wave;
    if (kc >= a.Nc) return;
    const int E = WHOLE ? EC : a.L / 64;
    const bool is_exp = a.variant == 0;
    const long row = (long)bh * a.T;
    AT* tb = reinterpret_cast<AT*>(a.tmp) + (long)bh * 3 * a.T;
    AT* tc = tb + a.T;
    AT* ta = tc + a.T;
    AT* csum = reinterpret_cast<AT*>(a.csum);
    const AT log2e = (AT)1.4426950408889634;
    const long t0 = (long)kc * a.L + (long)lane * E;
    // log gates of step t; the padding steps of a sequence that does not fill its last chunk keep the
    // state as it is (log forget gate 0) and add nothing (log input gate far below every other)
    const long urow = (long)bh * a.Tvalid;          // the caller's tensors
    auto fbar_at = [&](long t) { return t < a.Tvalid ? log_sigmoid_t<AT>(soft_cap_t<AT>((AT)a.f_pre[urow + t], a.softcap)) : (AT)0; };
    auto ibar_at = [&](long t) {
        if (t >= a.Tvalid) return (AT)-1.0e30f;
        const AT ip = soft_cap_t<AT>((AT)a.i_pre[urow + t], a.softcap);
        return is_exp ? ip : log_sigmoid_t<AT>(ip);
    };
    constexpr int NC = EC > 0 ? EC : 1;
    AT fbv[NC], ibv[NC];
    if constexpr (EC > 0) {
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            fbv[e] = (AT)0; ibv[e] = (AT)0;
            if (e < E) { fbv[e] = fbar_at(t0 + e); ibv[e] = ibar_at(t0 + e); }
        }
    }
    auto fbar = [&](int e) { if constexpr (EC > 0) return fbv[e]; else return fbar_at(t0 + e); };
    auto ibar = [&](int e) { if constexpr (EC > 0) return ibv[e]; else return ibar_at(t0 + e); };
    const int EB = EC > 0 ? EC : E;                 // loop bound (compile-time when the gates are cached)
    AT fsum = (AT)0;
#pragma unroll
    for (int e = 0; e < EB; ++e)
        if (e < E) fsum += fbar(e);
    AT gsum;
    const AT off = wave_excl_scan_add<AT>(fsum, lane, &gsum);
    const AT roff = wave_excl_rscan_add<AT>(fsum, lane);
    // forward pass: b, u = i-bar - b, running max of u
    AT b = off, cmx = (AT)-INFINITY;
#pragma unroll
    for (int e = 0; e < EB; ++e)
        if (e < E) {
            b += fbar(e);
            cmx = max_t<AT>(cmx, ibar(e) - b);
        }
    const AT cmoff = wave_excl_scan_max<AT>(cmx, lane);
    b = off; cmx = cmoff;
    AT bv[NC], cv[NC], av_[NC];
    float uhv[NC], ulv[NC];
#pragma unroll
    for (int e = 0; e < EB; ++e)
        if (e < E) {
            b += fbar(e);
            const AT u = ibar(e) - b;
            cmx = max_t<AT>(cmx, u);
            const AT ul = u * log2e;
            const float uh = (float)ul;
            if constexpr (WHOLE) {
                bv[e] = b; cv[e] = cmx; uhv[e] = uh; ulv[e] = (float)(ul - (AT)uh);
            } else {
                tb[t0 + e] = b;
                tc[t0 + e] = cmx;
                a.ucol[row + t0 + e] = uh;
                if (a.ucol_lo) a.ucol_lo[row + t0 + e] = (float)(ul - (AT)uh);
            }
        }
    // reverse pass: a_j = sum_{s>j} f-bar_s + i-bar_j
    AT run = roff, amax = (AT)-INFINITY;
#pragma unroll
    for (int e = EB - 1; e >= 0; --e)
        if (e < E) {
            const AT av = run + ibar(e);
            if constexpr (WHOLE) av_[e] = av;
            else ta[t0 + e] = av;
            amax = max_t<AT>(amax, av);
            run += fbar(e);
        }
    if constexpr (WHOLE) {
        store_steps<EC>(tb + t0, bv);
        store_steps<EC>(tc + t0, cv);
        store_steps<EC>(ta + t0, av_);
        store_steps<EC>(a.ucol + row + t0, uhv);
        if (a.ucol_lo) store_steps<EC>(a.ucol_lo + row + t0, ulv);
    }
    amax = wave_max_t<AT>(amax);
    if (lane == 0) {
        csum[((long)bh * 2 + 0) * a.Nc + kc] = gsum;
        csum[((long)bh * 2 + 1) * a.Nc + kc] = amax;
    }
}

// EC > 0: a lane has exactly EC steps, which move as vectors and are requested before the recurrence over the chunks
template <int EC, typename AT>
__global__ void __launch_bounds__(GATE_WAVES * 64) gates_step_kernel(GateArgs a) {
    if (a.variant != 0) zero_share(a.zero, ((long)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x, (long)gridDim.x * gridDim.y * blockDim.x);
    extern __shared__ double cm_raw[];   // [Nc + 1] values of type AT: m before chunk k
    AT* cm = reinterpret_cast<AT*>(cm_raw);
    const int bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool is_exp = a.variant == 0;
    const AT* cg = reinterpret_cast<const AT*>(a.csum) + ((long)bh * 2 + 0) * a.Nc;
    const AT* camax = reinterpret_cast<const AT*>(a.csum) + ((long)bh * 2 + 1) * a.Nc;
    const int kc = blockIdx.x * GATE_WAVES + wave;
    const int E = EC > 0 ? EC : a.L / 64;
    const long row = (long)bh * a.T;
    const AT* tb = reinterpret_cast<const AT*>(a.tmp) + (long)bh * 3 * a.T;
    const AT* tc = tb + a.T;
    const AT* ta = tc + a.T;
    const long t0 = (long)kc * a.L + (long)lane * E;
    constexpr int NC = EC > 0 ? EC : 1;
    AT bv[NC], cv[NC], av_[NC];
    if constexpr (EC > 0)
        if (kc < a.Nc) { load_steps<EC>(bv, tb + t0); load_steps<EC>(cv, tc + t0); load_steps<EC>(av_, ta + t0); }
    if (wave == 0) {
        // lane l composes the maps of its segment of chunks, a wavefront scan composes the segments,
        // then every lane walks its segment again from its incoming m
        const int seg = (a.Nc + 63) / 64;
        const int k0 = lane * seg, k1 = min(a.Nc, k0 + seg);
        AT G = (AT)0, C = (AT)-INFINITY;
        for (int k = k0; k < k1; ++k) { C = max_t<AT>(C + cg[k], camax[k]); G += cg[k]; }
        // exclusive scan over the lanes: the map of all chunks before this lane's segment, applied to m0
        struct Map { AT g, c; };
        const auto then = [](Map p, Map q) { return Map{p.g + q.g, max_t<AT>(p.c + q.g, q.c)}; };       // q after p
        const auto moved = [](Map p, auto ctrl) { return Map{row_move<decltype(ctrl)::value>(p.g, (AT)0), row_move<decltype(ctrl)::value>(p.c, (AT)-INFINITY)}; };
        const auto at = [](Map p, int l) { return Map{lane_value(p.g, l), lane_value(p.c, l)}; };
        Map x{G, C};
        x = then(moved(x, std::integral_constant<int, 0x111>()), x);
        x = then(moved(x, std::integral_constant<int, 0x112>()), x);
        x = then(moved(x, std::integral_constant<int, 0x114>()), x);
        x = then(moved(x, std::integral_constant<int, 0x118>()), x);
        const Map p0 = at(x, 15), p1 = then(p0, at(x, 31)), p2 = then(p1, at(x, 47));
        Map before{(AT)0, (AT)-INFINITY};
        if (lane >= 16) before = lane < 32 ? p0 : lane < 48 ? p1 : p2;
        before = then(before, moved(x, std::integral_constant<int, 0x111>()));
        const AT Ge = before.g, Ce = before.c;
        const AT m_init = (is_exp && a.m0) ? (AT)a.m0[bh] : (AT)0;
        AT m = lane == 0 ? m_init : max_t<AT>(m_init + Ge, Ce);
        if (!is_exp) m = (AT)0;
        for (int k = k0; k < k1; ++k) {
            cm[k] = m;
            const AT mn = is_exp ? max_t<AT>(cg[k] + m, camax[k]) : (AT)0;
            if (blockIdx.x == 0) a.gbar[(long)bh * a.Nc + k] = (float)exp_t<AT>(cg[k] + m - mn);
            m = mn;
        }
        if (k1 == a.Nc && k0 < k1) {
            cm[a.Nc] = m;
            if (blockIdx.x == 0 && a.mfinal) a.mfinal[bh] = (float)m;
        }
    }
    __syncthreads();
    if (kc >= a.Nc) return;
    const AT log2e = (AT)1.4426950408889634;
    const AT lq = (AT)log2f(a.qscale);
    const AT mprev = cm[kc], mk = cm[kc + 1];
    auto step = [&](AT b, AT cmx, AT av, float& wh, float& wl, float& shf, float& ak, float& mof) {
        AT wr, sh, mo;
        if (is_exp) {
            const AT M = max_t<AT>(mprev, cmx);
            wr = -M * log2e + lq;
            sh = exp_t<AT>(mprev - M) * (AT)a.qscale;
            mo = b + M;
        } else {
            wr = b * log2e + lq;
            sh = exp_t<AT>(b) * (AT)a.qscale;
            mo = (AT)0;
        }
        wh = (float)wr;
        wl = (float)(wr - (AT)wh);
        shf = (float)sh;
        ak = (float)exp_t<AT>(av - mk);
        mof = (float)mo;
    };
    if constexpr (EC > 0) {
        float wh[EC], wl[EC], sh[EC], ak[EC], mo[EC];
#pragma unroll
        for (int e = 0; e < EC; ++e) step(bv[e], cv[e], av_[e], wh[e], wl[e], sh[e], ak[e], mo[e]);
        store_steps<EC>(a.wrow + row + t0, wh);
        if (a.wrow_lo) store_steps<EC>(a.wrow_lo + row + t0, wl);
        store_steps<EC>(a.sH + row + t0, sh);
        store_steps<EC>(a.aK + row + t0, ak);
        store_steps<EC, 4>(a.mout + row + t0, mo);          // (may be the caller's tensor)
        if (a.mout_user) {
#pragma unroll
            for (int e = 0; e < EC; ++e)
                if (t0 + e < a.Tvalid) a.mout_user[(long)bh * a.Tvalid + t0 + e] = mo[e];
        }
    } else {
        for (int e = 0; e < E; ++e) {
            float wh, wl, sh, ak, mo;
            step(tb[t0 + e], tc[t0 + e], ta[t0 + e], wh, wl, sh, ak, mo);
            a.wrow[row + t0 + e] = wh;
            if (a.wrow_lo) a.wrow_lo[row + t0 + e] = wl;
            a.sH[row + t0 + e] = sh;
            a.aK[row + t0 + e] = ak;
            a.mout[row + t0 + e] = mo;
            if (a.mout_user && t0 + e < a.Tvalid) a.mout_user[(long)bh * a.Tvalid + t0 + e] = mo;
        }
    }
}

// Both kernels in one for short sequences (gates_in_one_launch): up to sixteen chunks, one wavefront each, in one workgroup per (batch, head);
// the lane's E = L / 64 steps stay in registers from the scans to the results, and the chunk summaries meet in LDS.
// Longer sequences keep the two launches, which spread one (batch, head) over the chip (a workgroup that walks 32 chunks
// twice took 34 us where the two take 16).  us, two launches / one: 8 heads of 8 chunks of 128 11 / 5.6; 256 heads of 8
// chunks of 256 23 / 12; 16 heads of 16 chunks of 256 17 / 13.
// The chunk sizes are those that give a lane 1, 2, 4 or 8 steps, one vector store per result; the others (192, 320, 1024, ...)
// keep the two launches as well.
template <int E, typename AT>
__global__ void __launch_bounds__(GATE_FUSED_CHUNKS * 64) gates_fused_kernel(GateArgs a) {
    if (a.variant != 0) zero_share(a.zero, (long)blockIdx.x * blockDim.x + threadIdx.x, (long)gridDim.x * blockDim.x);
    __shared__ AT cg[GATE_FUSED_CHUNKS], camax[GATE_FUSED_CHUNKS], m_init;
    const int bh = blockIdx.x, lane = threadIdx.x & 63, kc = threadIdx.x >> 6;
    const bool is_exp = a.variant == 0;
    const int t0 = kc * (64 * E) + lane * E;                       // first of this lane's steps
    const long row = (long)bh * a.T + t0, urow = (long)bh * a.Tvalid + t0;
    const AT log2e = (AT)1.4426950408889634;
    AT fb[E], ib[E], b[E], cm[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        fb[e] = (AT)0; ib[e] = (AT)-1.0e30f;                       // (a step past the end of the sequence)
        if (t0 + e < a.Tvalid) {
            fb[e] = log_sigmoid_t<AT>(soft_cap_t<AT>((AT)a.f_pre[urow + e], a.softcap));
            const AT ip = soft_cap_t<AT>((AT)a.i_pre[urow + e], a.softcap);
            ib[e] = is_exp ? ip : log_sigmoid_t<AT>(ip);
        }
    }
    AT fsum = (AT)0;
#pragma unroll
    for (int e = 0; e < E; ++e) fsum += fb[e];
    AT gsum;
    const AT off = wave_excl_scan_add<AT>(fsum, lane, &gsum), roff = wave_excl_rscan_add<AT>(fsum, lane);
    AT run = off, cmx = (AT)-INFINITY;
    float uh[E], ul[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        run += fb[e];
        b[e] = run;
        const AT u = ib[e] - run;
        cmx = max_t<AT>(cmx, u);
        cm[e] = cmx;
        uh[e] = (float)(u * log2e);
        ul[e] = (float)(u * log2e - (AT)uh[e]);
    }
    const AT cmoff = wave_excl_scan_max<AT>(cmx, lane);
    // a_j = sum_{s>j} f-bar_s + i-bar_j
    AT av[E], amax = (AT)-INFINITY;
    run = roff;
#pragma unroll
    for (int e = E - 1; e >= 0; --e) {
        av[e] = run + ib[e];
        amax = max_t<AT>(amax, av[e]);
        run += fb[e];
    }
    amax = wave_max_t<AT>(amax);
    if (lane == 0) { cg[kc] = gsum; camax[kc] = amax; }
    // (read once, before the barrier: the caller's final state may be the buffer of its initial state, and the last chunk's
    // wavefront writes it without waiting for the others)
    if (threadIdx.x == 0) m_init = (is_exp && a.m0) ? (AT)a.m0[bh] : (AT)0;
    __syncthreads();
    AT mprev = m_init;
    if (is_exp)
        for (int k = 0; k < kc; ++k) mprev = max_t<AT>(cg[k] + mprev, camax[k]);
    const AT mk = is_exp ? max_t<AT>(gsum + mprev, amax) : (AT)0;
    if (lane == 0) {
        a.gbar[(long)bh * a.Nc + kc] = (float)exp_t<AT>(gsum + mprev - mk);
        if (kc == a.Nc - 1 && a.mfinal) a.mfinal[bh] = (float)mk;
    }
    const AT lq = (AT)log2f(a.qscale);
    typedef float vec __attribute__((ext_vector_type(E)));
    vec wh, wl, sh, ak, uv, uvl;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        AT wr, s, mo = (AT)0;
        if (is_exp) {
            const AT M = max_t<AT>(mprev, max_t<AT>(cmoff, cm[e]));
            wr = -M * log2e + lq;
            s = exp_t<AT>(mprev - M) * (AT)a.qscale;
            mo = b[e] + M;
        } else {
            wr = b[e] * log2e + lq;
            s = exp_t<AT>(b[e]) * (AT)a.qscale;
        }
        wh[e] = (float)wr; wl[e] = (float)(wr - (AT)wh[e]);
        sh[e] = (float)s;
        ak[e] = (float)exp_t<AT>(av[e] - mk);
        uv[e] = uh[e]; uvl[e] = ul[e];
        a.mout[row + e] = (float)mo;
        if (a.mout_user && t0 + e < a.Tvalid) a.mout_user[urow + e] = (float)mo;
    }
    *reinterpret_cast<vec*>(a.wrow + row) = wh;
    *reinterpret_cast<vec*>(a.ucol + row) = uv;
    *reinterpret_cast<vec*>(a.sH + row) = sh;
    *reinterpret_cast<vec*>(a.aK + row) = ak;
    if (a.wrow_lo) *reinterpret_cast<vec*>(a.wrow_lo + row) = wl;
    if (a.ucol_lo) *reinterpret_cast<vec*>(a.ucol_lo + row) = uvl;
}

template <typename AT> static hipError_t launch_gates_t(const GateArgs& a, int BH, hipStream_t s) {
    if (gates_in_one_launch(a.Nc, a.L)) {
        const dim3 grid(BH), block(64 * a.Nc);
        if (a.L == 64) hipLaunchKernelGGL((gates_fused_kernel<1, AT>), grid, block, 0, s, a);
        else if (a.L == 128) hipLaunchKernelGGL((gates_fused_kernel<2, AT>), grid, block, 0, s, a);
        else if (a.L == 256) hipLaunchKernelGGL((gates_fused_kernel<4, AT>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((gates_fused_kernel<8, AT>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    const dim3 grid((a.Nc + GATE_WAVES - 1) / GATE_WAVES, BH);
    const dim3 block(GATE_WAVES * 64);
    const size_t lds = sizeof(AT) * (size_t)(a.Nc + 1);
    auto both = [&](auto chunk_kernel, auto step_kernel) {
        hipLaunchKernelGGL(chunk_kernel, grid, block, 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(step_kernel, grid, block, lds, s, a);
        return hipGetLastError();
    };
    // the log gates of a lane's steps stay in registers for every chunk size the library accepts (L <= 2048)
    switch (a.L) {
        case 64: return both(gates_chunk_kernel<1, AT, true>, gates_step_kernel<1, AT>);
        case 128: return both(gates_chunk_kernel<2, AT, true>, gates_step_kernel<2, AT>);
        case 256: return both(gates_chunk_kernel<4, AT, true>, gates_step_kernel<4, AT>);
        case 512: return both(gates_chunk_kernel<8, AT, true>, gates_step_kernel<8, AT>);
    }
    if (a.L / 64 <= 8) return both(gates_chunk_kernel<8, AT, false>, gates_step_kernel<0, AT>);
    if (a.L / 64 <= 16) return both(gates_chunk_kernel<16, AT, false>, gates_step_kernel<0, AT>);
    if (a.L / 64 <= 32) return both(gates_chunk_kernel<32, AT, false>, gates_step_kernel<0, AT>);
    return both(gates_chunk_kernel<0, AT, false>, gates_step_kernel<0, AT>);
}

// a.precise: the fp32 kernels' pre-pass (double arithmetic, two-float exponents; tmp and csum then hold doubles)
hipError_t launch_gates(const GateArgs& a, int BH, hipStream_t s) {
    return a.precise ? launch_gates_t<double>(a, BH, s) : launch_gates_t<float>(a, BH, s);
}

// Backward preparation: fold delta H~ = delta H / h_denom (App. B.3) into the weights.
__global__ void gate_bwd_prep_kernel(GateBwdPrepArgs a) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    float den = 1.0f;
    if (a.variant == 0) {
        long u = i;
        bool there = true;
        if (a.Tvalid != a.T) {          // (steps past the end of the sequence: any finite non-zero value would do)
            const long bh = i / a.T, t = i - bh * a.T;
            there = t < a.Tvalid;
            u = bh * a.Tvalid + t;
        }
        if (there) den = fmaxf(fabsf(a.n_out[u]), expf(-a.m_out[u])) + a.eps;
    }
    if (a.wrowB_lo) {
        // fp32 kernels: the difference to double accuracy, as a (rounded, remainder) pair
        const double w = (double)a.wrow[i] + (double)a.wrow_lo[i] - log2((double)den);
        const float wh = (float)w;
        a.wrowB[i] = wh;
        a.wrowB_lo[i] = (float)(w - (double)wh);
    } else {
        a.wrowB[i] = a.wrow[i] - log2f(den);
    }
    a.sQ[i] = a.sH[i] / den;
}
hipError_t launch_gate_bwd_prep(const GateBwdPrepArgs& a, hipStream_t s) {
    const int nt = 256;
    hipLaunchKernelGGL(gate_bwd_prep_kernel, dim3((unsigned)((a.n + nt - 1) / nt)), dim3(nt), 0, s, a);
    return hipGetLastError();
}

// Gate gradients.  q_t . dq_t and k_t . dk_t are the row and column sums of the gradient
// w.r.t. the log weights (each log weight is linear in the f-bar_s it spans and in i-bar_j), so
//   d i-bar_j = k_j . dk_j ,   d f-bar_s = sum_{t>=s} (q_t . dq_t - k_t . dk_t) + <C_T, dC_T>.
// This regroups the cumulative-gate gradients of App. B.3 (delta g, delta a, delta b and the
// row/column sums of the intra-chunk gate-matrix gradient) into one reverse cumulative sum.
// Over blocks of GG_BLOCK steps: every block adds the sums of the blocks after it and scans its own steps (in fp64: the
// terms cancel heavily).  Up to GG_ONE blocks the block forms those sums itself; beyond, a launch before it leaves them
// in memory once (the launch is 4 to 7 us, the terms of three blocks are read in one).
static constexpr int GG_BLOCK = 1024, GG_ONE = 4;

__device__ __forceinline__ double state_dot_sum(const GateGradArgs& a, int bh) {
    double s = 0.0;
    if (a.cdot) {
#pragma unroll
        for (int p = 0; p < STATE_DOT_PARTS; ++p) s += a.cdot[(long)bh * STATE_DOT_PARTS + p];
    }
    return s;
}
__device__ __forceinline__ void gate_grad_terms(const GateGradArgs& a, long idx, float& r, float& c) {
    r = 0.0f; c = 0.0f;
    for (int nb = 0; nb < a.nbQ; ++nb) r += a.partQ[(long)nb * a.BHT + idx];
    for (int nb = 0; nb < a.nbK; ++nb) c += a.partK[(long)nb * a.BHT + idx];
}

// this thread's part of the sum over block blk
__device__ __forceinline__ double gate_grad_block_part(const GateGradArgs& a, long row, int blk, int tid) {
    double tot = 0.0;
#pragma unroll
    for (int e = 0; e < GG_BLOCK / 256; ++e) {
        const int t = blk * GG_BLOCK + e * 256 + tid;
        if (t < a.T) {
            float r, c;
            gate_grad_terms(a, row + t, r, c);
            tot += (double)r - (double)c;
        }
    }
    return tot;
}

__global__ void __launch_bounds__(256) gate_grads_sum_kernel(GateGradArgs a) {
    __shared__ double wt[4];
    const int bh = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
    const double tot = wave_sum_t<double>(gate_grad_block_part(a, (long)bh * a.T, blk, tid));
    if ((tid & 63) == 0) wt[tid >> 6] = tot;
    __syncthreads();
    if (tid == 0) a.bsum[(long)bh * gridDim.x + blk] = wt[0] + wt[1] + wt[2] + wt[3];
}

__global__ void __launch_bounds__(256) gate_grads_kernel(GateGradArgs a) {
    __shared__ double wt[4];
    __shared__ double after;
    const int bh = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nblk = gridDim.x;
    const long row = (long)bh * a.T;
    // sum of the blocks after this one
    double later = 0.0;
    if (nblk <= GG_ONE) {
        for (int b2 = blk + 1; b2 < nblk; ++b2) later += gate_grad_block_part(a, row, b2, tid);
    } else {
        for (int b2 = blk + 1 + tid; b2 < nblk; b2 += 256) later += a.bsum[(long)bh * nblk + b2];
    }
    later = wave_sum_t<double>(later);
    if (lane == 0) wt[wave] = later;
    __syncthreads();
    if (tid == 0) after = wt[0] + wt[1] + wt[2] + wt[3] + state_dot_sum(a, bh);
    __syncthreads();
    // thread tid owns GG_BLOCK / 256 consecutive steps
    constexpr int SEG = GG_BLOCK / 256;
    const int t0 = blk * GG_BLOCK + tid * SEG;
    float r[SEG], c[SEG];
    double tot = 0.0;
#pragma unroll
    for (int e = 0; e < SEG; ++e) {
        r[e] = 0.0f; c[e] = 0.0f;
        if (t0 + e < a.T) gate_grad_terms(a, row + t0 + e, r[e], c[e]);
        tot += (double)r[e] - (double)c[e];
    }
    double excl = wave_excl_rscan_add<double>(tot, lane);
    __syncthreads();
    if (lane == 0) wt[wave] = tot + excl;
    __syncthreads();
    for (int w = wave + 1; w < 4; ++w) excl += wt[w];
    double run = excl + after;
#pragma unroll
    for (int e = SEG - 1; e >= 0; --e) {
        const int t = t0 + e;
        if (t < a.T) {
            run += (double)r[e] - (double)c[e];
            if (t < a.Tvalid) {
                const long u = (long)bh * a.Tvalid + t;
                const float fp = a.f_pre[u], ip = a.i_pre[u];
                a.d_f[u] = (float)run * sigmoid_neg(soft_cap(fp, a.softcap)) * soft_cap_grad(fp, a.softcap);
                a.d_i[u] = (a.variant == 0 ? c[e] : c[e] * sigmoid_neg(soft_cap(ip, a.softcap))) * soft_cap_grad(ip, a.softcap);
            }
        }
    }
}
// The same with anchors.  The value of the reverse cumulative sum at a chunk boundary is known exactly:
// the log forget gate of the first step of chunk k + 1 scales the boundary state C_{k+1} in every later
// use, so d f-bar there is <C_{k+1}, dC_{k+1}>, which needs no summation over time.  Every block of G chunks
// then scans its own steps only, from the anchor at its end, and the rounding noise of the terms no longer
// accumulates over the whole sequence (it grows with sqrt(T) in the unanchored scan).  One workgroup per
// block (at most 4096 steps, ANCHOR_STEPS); a thread owns up to sixteen consecutive steps.
// SC > 0: a thread owns exactly SC steps (a block is 256 SC steps), whose terms move as vectors; 0: any number up to MOST.
template <int SC, int MOST = SC>
__global__ void __launch_bounds__(256) gate_grads_anchored_kernel(GateGradArgs a) {
    __shared__ double wt[4];
    const int bh = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long row = (long)bh * a.T;
    const int kc0 = blk * a.G, kc1 = min(kc0 + a.G, a.Nc);      // chunks [kc0, kc1)
    const long tb = (long)kc0 * a.L;                            // first step of the block
    const int len = (kc1 - kc0) * a.L;                          // steps in this block
    const int SEG = SC > 0 ? SC : (a.G * a.L + 255) / 256;     // <= MOST: the launcher's rule
    constexpr int NE = MOST;
    const int l0 = tid * SEG;                          // first of this thread's steps within the block
    float r[NE], c[NE], fpre[NE], ipre[NE];
    double tot = 0.0;
    // (the gate pre-activations are requested ahead of the scan)
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const bool there = e < SEG && l0 + e < len && tb + l0 + e < a.Tvalid;
        const long u = (long)bh * a.Tvalid + tb + l0 + e;
        fpre[e] = there ? a.f_pre[u] : 0.0f;
        ipre[e] = there ? a.i_pre[u] : 0.0f;
    }
    if constexpr (SC > 0) {
#pragma unroll
        for (int e = 0; e < NE; ++e) { r[e] = 0.0f; c[e] = 0.0f; }
        if (l0 < len) {             // (whole segments: len is a multiple of SC)
            float v[SC];
            for (int nb = 0; nb < a.nbQ; ++nb) {
                load_steps<SC>(v, a.partQ + (long)nb * a.BHT + row + tb + l0);
#pragma unroll
                for (int e = 0; e < SC; ++e) r[e] += v[e];
            }
            for (int nb = 0; nb < a.nbK; ++nb) {
                load_steps<SC>(v, a.partK + (long)nb * a.BHT + row + tb + l0);
#pragma unroll
                for (int e = 0; e < SC; ++e) c[e] += v[e];
            }
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) tot += (double)r[e] - (double)c[e];
    } else {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            r[e] = 0.0f; c[e] = 0.0f;
            if (e < SEG && l0 + e < len) gate_grad_terms(a, row + tb + l0 + e, r[e], c[e]);
            tot += (double)r[e] - (double)c[e];
        }
    }
    double excl = wave_excl_rscan_add<double>(tot, lane);
    if (lane == 0) wt[wave] = tot + excl;
    __syncthreads();
    for (int w = wave + 1; w < 4; ++w) excl += wt[w];
    // the anchor at the end of the block: <C_T, dC_T> (or nothing) at the end of the sequence, else <C, dC> at the
    // boundary after the block, which the reversed recurrent launch left as npart partial sums
    __shared__ double wa[4];
    double anc = 0.0;
    if (kc1 == a.Nc) {
        anc = state_dot_sum(a, bh);
    } else {
        const int nslot = (a.Nc + a.G - 1) / a.G;
        const float* pp = a.anchor + ((long)bh * nslot + kc1 / a.G) * a.npart;
        double ps = 0.0;
        for (int q = tid; q < a.npart; q += 256) ps += (double)pp[q];
        ps = wave_sum_t<double>(ps);
        if (lane == 0) wa[wave] = ps;
        __syncthreads();
        anc = (wa[0] + wa[1]) + (wa[2] + wa[3]);
    }
    double run = excl + anc;
#pragma unroll
    for (int e = NE - 1; e >= 0; --e) {
        if (e < SEG && l0 + e < len) {
            const long t = tb + l0 + e;
            run += (double)r[e] - (double)c[e];
            if (t < a.Tvalid) {
                const long u = (long)bh * a.Tvalid + t;
                const float fp = fpre[e], ip = ipre[e];
                a.d_f[u] = (float)run * sigmoid_neg(soft_cap(fp, a.softcap)) * soft_cap_grad(fp, a.softcap);
                a.d_i[u] = (a.variant == 0 ? c[e] : c[e] * sigmoid_neg(soft_cap(ip, a.softcap))) * soft_cap_grad(ip, a.softcap);
            }
        }
    }
}

hipError_t launch_gate_grads(const GateGradArgs& a, int BH, hipStream_t s) {
    if (a.anchor) {
        if (a.G < 1 || (long)a.G * a.L > ANCHOR_STEPS) return hipErrorInvalidValue;
        const dim3 grid((a.Nc + a.G - 1) / a.G, BH);
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, a); };
        switch (a.G * a.L) {
            case 256: launch(gate_grads_anchored_kernel<1>); break;
            case 512: launch(gate_grads_anchored_kernel<2>); break;
            case 1024: launch(gate_grads_anchored_kernel<4>); break;
            case 2048: launch(gate_grads_anchored_kernel<8>); break;
            default:
                if (a.G * a.L < 2048) launch(gate_grads_anchored_kernel<0, 8>);
                else launch(gate_grads_anchored_kernel<0, ANCHOR_STEPS / 256>);     // (heads wider than 512, chunks above 1024)
        }
        return hipGetLastError();
    }
    const dim3 grid((a.T + GG_BLOCK - 1) / GG_BLOCK, BH);
    if (grid.x > GG_ONE) {
        hipLaunchKernelGGL(gate_grads_sum_kernel, grid, dim3(256), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(gate_grads_kernel, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

// (the shares stride through the arrays: any number of workgroups does)
__global__ void __launch_bounds__(256) zero_kernel(FillList f) { zero_share(f, (long)blockIdx.x * 256 + threadIdx.x, (long)gridDim.x * 256); }
hipError_t launch_zero(const FillList& f, hipStream_t s) {
    hipLaunchKernelGGL(zero_kernel, dim3(256), dim3(256), 0, s, f);
    return hipGetLastError();
}
__global__ void __launch_bounds__(256) copy_kernel(const float* from, float* to, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) to[i] = from[i];
}
hipError_t launch_copy(const float* from, float* to, int n, hipStream_t s) {
    hipLaunchKernelGGL(copy_kernel, dim3((n + 255) / 256), dim3(256), 0, s, from, to, n);
    return hipGetLastError();
}
// Part p of <A[bh], Bm[bh]> over the d1 x d2 values of Bm (A's rows are lda apart): rows p, p + STATE_DOT_PARTS, ...,
// the wavefronts of the workgroup one row each.  (One workgroup per (batch, head) took 17 us for 32 heads of 96 x 192, 12
// us for 16 of 128 x 256; now 6 and 6.)
__global__ void __launch_bounds__(256) state_dot_kernel(const float* A, long perA, int lda, const float* Bm, int d1, int d2, double* out) {
    __shared__ double wt[4];
    const int bh = blockIdx.y, p = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double acc = 0.0;
    for (int r = p + STATE_DOT_PARTS * wave; r < d1; r += 4 * STATE_DOT_PARTS) {
        const float* ar = A + bh * perA + (long)r * lda;
        const float* br = Bm + ((long)bh * d1 + r) * d2;
        for (int c = lane; c < d2; c += 64) acc += (double)ar[c] * (double)br[c];
    }
    acc = wave_sum_t<double>(acc);
    if (lane == 0) wt[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[(long)bh * STATE_DOT_PARTS + p] = (wt[0] + wt[1]) + (wt[2] + wt[3]);
}
hipError_t launch_state_dot(const float* A, long perA, int lda, const float* Bm, int d1, int d2, double* out, int BH, hipStream_t s) {
    hipLaunchKernelGGL(state_dot_kernel, dim3(STATE_DOT_PARTS, BH), dim3(256), 0, s, A, perA, lda, Bm, d1, d2, out);
    return hipGetLastError();
}

}  // namespace tfla
