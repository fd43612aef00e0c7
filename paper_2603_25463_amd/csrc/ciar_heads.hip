// gfx950 kernels for several Interval Heads (Sec. 4, ablation on the Inter-Head): the Ensemble sweep that
// averages the heads' widths token by token, and the Voting majority.
#include "ciar_device.h"

#include <mutex>
#include <type_traits>

namespace ciar {
namespace {

// ---- several heads (Sec. 4, ablation on the Inter-Head): Ensemble and Voting ------------------------------

constexpr int kMaxHeads = 8;

// Ensemble: the heads' curves are averaged token by token, so the widths of all heads of a token have to
// meet: a second sweep over the H rows of a position, after the streaming kernel has left every head's
// RowStats (partition sum, reference, interval sums -> that head's caps).  One workgroup per position;
// per token and head the same arithmetic as the streaming kernel's interval pass.
//   D_i = sum_h delta_{h,i},  Omega = sum_i D_i / H,  Sigma^2 = sum_i D_i^2 / (H^2 V) - (Omega / V)^2.
// WIDE (calls with a wide radius, see wide_radius): also C_i = sum_h (1 - width_{h,i}); where every mean width is
// above 1/2 and no head has an active cap, D_i = H - C_i, and Omega and Sigma are taken from the sums of C_i,
// which resolve a spread that the widths, all rounding to 1, no longer show.
template <typename T, bool WIDE>
__global__ __launch_bounds__(256) void ensemble_kernel(const RowArgs A, const int H, const int64_t head_stride)
{
    using E = Elt<T>;
    constexpr int EPV = E::kPerVec;
    __shared__ FuseRow sm_fr[kMaxHeads];
    __shared__ float sm_n[kMaxHeads], sm_invS[kMaxHeads];
    __shared__ double sm_cw[kMaxHeads], sm_cl[kMaxHeads], sm_S[kMaxHeads], sm_al[kMaxHeads], sm_au[kMaxHeads];
    __shared__ double sm_red[5][4];
    __shared__ float sm_pm[4];
    __shared__ int sm_pi[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;
    const int V = A.V;
    const bool rad = A.radius != nullptr;
    const bool need_argmax = A.ids == nullptr && (A.p_lo || A.p_mid || A.p_hi);
    bool flat_h = true;                                            // this lane's head: a flat row (see below)
    if (tid < H) {
        const RowStats st = A.stats[(int64_t)tid * A.N + row];
        flat_h = (double)Elt<T>::exp2_ref(st.mc, st.n == -INFINITY ? 0.f : st.n) * (double)V <= 2.0 * st.S;
        const RowScore rs = finish_score(st.q, st.S, st.mode, A, st.kl, st.kw);
        const double Bc = (rad ? 1.0 : A.b) / st.S, Wc = (rad ? 1.0 : A.a - A.b) / st.S;
        sm_fr[tid] = fuse_row(st.S, A.a, A.b);
        sm_n[tid] = st.n;
        sm_cw[tid] = rs.alpha_u * Wc;
        sm_cl[tid] = (rs.alpha_u - rs.alpha_l) * Bc;
        sm_invS[tid] = (float)(1.0 / st.S);
        sm_S[tid] = st.S; sm_al[tid] = rs.alpha_l; sm_au[tid] = rs.alpha_u;
    }
    // Token arithmetic in fp64 ("precise") for rows of a handful of tokens and for rows that are flat in every
    // head (largest probability <= 2 / V): there the widths can agree to 1e-4 and better while their fp32 errors
    // (~1e-7 each, uncorrelated when the radii differ from token to token) do not, and Omega ~ V multiplies what
    // is left of the spread.
    const bool precise = __syncthreads_and(flat_h ? 1 : 0) != 0 || V <= 64;   // uniform; also the barrier
    // no head with an active cap (delta = alpha_u w + (alpha_u - alpha_l) p^l loses its second term): uniform
    const bool no_lower = __syncthreads_and(tid < H ? (sm_cl[tid] == 0.0 ? 1 : 0) : 1) != 0;

    const RadiusMode rm = radius_mode(A);
    const int nvec = (V + EPV - 1) / EPV;
    // One head's share of a token: its width after the head's caps (added to d) and, WIDE, its complement (to c).
    auto head_token = [&](int h, float cval, float rval, const FuseRow& fr, double& d, double& c) {
        const float e = Elt<T>::exp2_ref(cval, sm_n[h]);
        float gl, gw;
        if constexpr (WIDE) {
            float ec;
            if (rad) fuse_token_rad_wide<T>(e, rval, fr, rm, gl, gw, ec);
            else fuse_token_wide(e, fr, gl, gw, ec);
            c += (double)ec;
        } else {
            if (rad) fuse_token_rad<T>(e, rval, fr, rm, gl, gw);
            else fuse_token(e, fr, gl, gw);
        }
        d = fma(sm_cw[h], (double)gw, fma(sm_cl[h], (double)gl, d));
        return e;
    };
    // The same in fp64 from the fp32 e (rows of a handful of tokens).
    auto head_token_tiny = [&](int h, float cval, float rval, double& d, double& c) {
        // A handful of tokens: e as the streaming kernel summed it into S, so that 1 - x stays accurate as x -> 1.
        // A flat row: the fp64 exponential (every x is tiny; the fp32 one would leave 6e-8 of each width behind,
        // uncorrelated from token to token, where the widths themselves agree to 1e-6).
        const double ed = V <= 64 ? (double)Elt<T>::exp2_ref(cval, sm_n[h]) : exp(ln_exp2<T>(cval, (double)sm_n[h]));
        const double x = ed / sm_S[h], omx = fmax(0.0, sm_S[h] - ed) / sm_S[h];
        double a = A.a, b = A.b;
        if (rad) {
            const double rr = radius_of((double)rval, A.kappa, A.rmax);
            a = exp(rr); b = exp(-rr);
        }
        const double du = 1.0 + (a - 1.0) * x, dl = b + (1.0 - b) * omx;
        d += sm_au[h] * a * x / du - sm_al[h] * b * x / dl;
        if constexpr (WIDE) c += (1.0 - 2.0 * (1.0 - b) * x * omx) / (du * dl);
        return x;
    };
    // The sums over the tokens are taken about D and C of the row's first token (every lane forms the same two
    // numbers): the spread of a row whose widths all agree is then 0 instead of the rounding noise that the
    // difference of two large moments leaves.
    double KD = 0.0, KC = 0.0;
    auto first_token = [&](bool in_fp64) {
        KD = 0.0; KC = 0.0;
        for (int h = 0; h < H; ++h) {
            const T* crow = static_cast<const T*>(A.draft) + (int64_t)h * head_stride + row * A.stride;
            const T* rrow = static_cast<const T*>(rad ? A.radius : A.draft) + (int64_t)h * head_stride + row * A.stride;
            const float c0 = load_logit(crow, 0), r0 = load_logit(rrow, 0);
            if (in_fp64) head_token_tiny(h, c0, r0, KD, KC);
            else head_token(h, c0, r0, sm_fr[h], KD, KC);
        }
    };
    first_token(precise);
    double s1 = 0.0, s2 = 0.0;                                     // sum (D_i - KD), sum (D_i - KD)^2
    double c1 = 0.0, c2 = 0.0, cbig = 0.0;                         // WIDE: sum (C_i - KC), its square, max C_i
    float best = -INFINITY;
    int best_i = INT_MAX;
    auto precise_sweep = [&]() {
        s1 = 0.0; s2 = 0.0; c1 = 0.0; c2 = 0.0; cbig = 0.0;
        best = -INFINITY; best_i = INT_MAX;
        for (int v = tid; v < nvec; v += 256) {
            double D[EPV], C[EPV];
            float pm[EPV];
#pragma unroll
            for (int k = 0; k < EPV; ++k) { D[k] = 0.0; C[k] = 0.0; pm[k] = 0.f; }
            for (int h = 0; h < H; ++h) {
                const gvec c = (gvec)(gbytes)(static_cast<const T*>(A.draft) + (int64_t)h * head_stride + row * A.stride);
                const gvec r = (gvec)(gbytes)(static_cast<const T*>(rad ? A.radius : A.draft) +
                                              (int64_t)h * head_stride + row * A.stride);
                const u32x4 cw4 = c[v], rw4 = r[v];
                float cv[EPV], rv[EPV];
                E::unpack(cw4, cv);
                E::unpack(rw4, rv);
                for (int k = 0; k < EPV; ++k) {
                    if (v * EPV + k < V) pm[k] += (float)head_token_tiny(h, cv[k], rv[k], D[k], C[k]);
                }
            }
            for (int k = 0; k < EPV; ++k) {
                const int tok = v * EPV + k;
                if (tok < V) {
                    const double d = D[k] - KD;
                    s1 += d;
                    s2 = fma(d, d, s2);
                    if constexpr (WIDE) {
                        const double c = C[k] - KC;
                        c1 += c; c2 = fma(c, c, c2); cbig = fmax(cbig, C[k]);
                    }
                }
                if (need_argmax && tok < V && pm[k] > best) { best = pm[k]; best_i = tok; }
            }
        }
    };
    if (precise) precise_sweep();
    // The sweep proper, specialised on what is uniform over the launch or the row: MODE bit 0 = tensor radius,
    // bit 1 = unit radius scale (see radius_am1), bit 2 = no head has an active cap (p^l is not needed).
    // Two 16-byte vectors of a head in flight per lane (fp32; one for bf16): more of them cost registers and
    // with them a wave per SIMD, which measured slower (four: +4 %, eight: +70 %).
    constexpr int UB = EPV >= 8 ? 1 : 8 / EPV;
    auto sweep = [&](auto mode_c) {
        constexpr int MODE = decltype(mode_c)::value;
        constexpr bool RADc = (MODE & 1) != 0, UNITc = (MODE & 2) != 0, NOLOW = (MODE & 4) != 0;
        for (int v0 = tid; v0 < nvec; v0 += 256 * UB) {
            double D[UB][EPV];                                     // fp64 across heads
            double C[WIDE ? UB : 1][EPV];
            float pm[UB][EPV];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    D[u][k] = 0.0; pm[u][k] = 0.f;
                    if constexpr (WIDE) C[u][k] = 0.0;
                }
            }
            for (int h = 0; h < H; ++h) {
                const gvec c = (gvec)(gbytes)(static_cast<const T*>(A.draft) + (int64_t)h * head_stride + row * A.stride);
                const gvec r = (gvec)(gbytes)(static_cast<const T*>(RADc ? A.radius : A.draft) +
                                              (int64_t)h * head_stride + row * A.stride);
                u32x4 cw4[UB], rw4[UB];
#pragma unroll
                for (int u = 0; u < UB; ++u) cw4[u] = c[min(v0 + u * 256, nvec - 1)];
                if constexpr (RADc) {
#pragma unroll
                    for (int u = 0; u < UB; ++u) rw4[u] = r[min(v0 + u * 256, nvec - 1)];
                }
                const FuseRow fr = sm_fr[h];
                const float invS = sm_invS[h], nh = sm_n[h];
                const double cw = sm_cw[h], cl = sm_cl[h];
                auto token = [&](float cval, float rval, double& d, double& cc, float& p) {
                    const float e = Elt<T>::exp2_ref(cval, nh);
                    float gl, gw;
                    if constexpr (WIDE) {
                        float ec;
                        if constexpr (RADc) fuse_token_rad_wide<T, UNITc>(e, rval, fr, rm.kappa, rm.rmax, rm.am1_max, gl, gw, ec);
                        else fuse_token_wide(e, fr, gl, gw, ec);
                        cc += (double)ec;
                    } else {
                        if constexpr (RADc) fuse_token_rad<T, UNITc>(e, rval, fr, rm.kappa, rm.rmax, rm.am1_max, gl, gw);
                        else fuse_token(e, fr, gl, gw);
                    }
                    if constexpr (NOLOW) d = fma(cw, (double)gw, d);
                    else d = fma(cw, (double)gw, fma(cl, (double)gl, d));
                    p = fmaf(e, invS, p);
                };
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    const int tok0 = (v0 + u * 256) * EPV;         // >= V for vectors past the row's end
                    float cv[EPV], rv[EPV];
                    E::unpack(cw4[u], cv);
                    if constexpr (RADc) E::unpack(rw4[u], rv);
                    if (tok0 + EPV <= V) {                         // a whole vector of tokens: no per-token test
#pragma unroll
                        for (int k = 0; k < EPV; ++k) token(cv[k], RADc ? rv[k] : 0.f, D[u][k], C[WIDE ? u : 0][k], pm[u][k]);
                    } else {
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            if (tok0 + k < V) token(cv[k], RADc ? rv[k] : 0.f, D[u][k], C[WIDE ? u : 0][k], pm[u][k]);
                        }
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    const int tok = (v0 + u * 256) * EPV + k;
                    if (tok < V) {
                        const double d = D[u][k] - KD;
                        s1 += d;
                        s2 = fma(d, d, s2);
                        if constexpr (WIDE) {
                            const double c = C[u][k] - KC;
                            c1 += c; c2 = fma(c, c, c2); cbig = fmax(cbig, C[u][k]);
                        }
                    }
                    if (need_argmax && tok < V && pm[u][k] > best) { best = pm[u][k]; best_i = tok; }
                }
            }
        }
    };
    if (!precise) {
        const int mode = (rad ? 1 : 0) | (rad && rm.unit ? 2 : 0) | (no_lower ? 4 : 0);
        switch (mode) {
        case 0: sweep(std::integral_constant<int, 0>{}); break;
        case 1: sweep(std::integral_constant<int, 1>{}); break;
        case 3: sweep(std::integral_constant<int, 3>{}); break;
        case 4: sweep(std::integral_constant<int, 4>{}); break;
        case 5: sweep(std::integral_constant<int, 5>{}); break;
        default: sweep(std::integral_constant<int, 7>{}); break;
        }
    }
    auto reduce = [&]() {
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if (lane == 0) { sm_red[0][wave] = s1; sm_red[1][wave] = s2; }
        if constexpr (WIDE) {
            c1 = wave_sum(c1);
            c2 = wave_sum(c2);
            cbig = (double)wave_max((float)cbig);
            if (lane == 0) { sm_red[2][wave] = c1; sm_red[3][wave] = c2; sm_red[4][wave] = cbig; }
        }
        if (need_argmax) {
            // each lane walked its tokens in ascending order, so it holds its lowest index of its maximum
            const float wm = wave_max(best);
            const int wi = wave_min_i(best == wm ? best_i : INT_MAX);
            if (lane == 0) { sm_pm[wave] = wm; sm_pi[wave] = wi; }
        }
        __syncthreads();
    };
    reduce();
    if (!precise) {
        // A row whose averaged widths agree to better than a hundredth of their mean although it is not flat in the
        // centre logits (heads whose widths crowd against 1 averaged with heads whose widths are next to nothing: every
        // D_i is about the same number): the ~1e-7 that fp32 token arithmetic leaves in each width is then no longer
        // small against the spread, and Omega multiplies what it does to Sigma (a seeded random case with a
        // tensor radius of scale 17: score off by 2e-5 of itself).  Such rows -- rare -- are swept again in fp64.
        // Every lane takes the same decision from the same numbers.
        const double t1 = (sm_red[0][0] + sm_red[0][1]) + (sm_red[0][2] + sm_red[0][3]);
        const double t2 = (sm_red[1][0] + sm_red[1][1]) + (sm_red[1][2] + sm_red[1][3]);
        const double Vd = (double)V, mean = (t1 + Vd * KD) / Vd, varD = fmax(0.0, t2 - t1 * t1 / Vd) / Vd;
        bool tight = varD < 1e-4 * mean * mean;
        if constexpr (WIDE) {
            // (not where the complement sums are read: they resolve exactly this case on their own)
            const double ub = fmax(fmax(sm_red[4][0], sm_red[4][1]), fmax(sm_red[4][2], sm_red[4][3]));
            bool plain = ub < kComplementBelow * (double)H;
            for (int h = 0; h < H; ++h) plain = plain && sm_al[h] == 1.0 && sm_au[h] == 1.0;
            tight = tight && !plain;
        }
        if (tight) {
            __syncthreads();                                       // sm_red is read by every lane above
            first_token(true);
            precise_sweep();
            reduce();
        }
    }
    if (tid == 0) {
        const double t1 = (sm_red[0][0] + sm_red[0][1]) + (sm_red[0][2] + sm_red[0][3]);
        const double t2 = (sm_red[1][0] + sm_red[1][1]) + (sm_red[1][2] + sm_red[1][3]);
        const double Hd = (double)H, Vd = (double)V;
        // t1 = sum (D_i - KD), t2 = sum (D_i - KD)^2
        double omega = (t1 + Vd * KD) / Hd;
        double var = fmax(0.0, t2 - t1 * t1 / Vd) / (Hd * Hd * Vd);
        if constexpr (WIDE) {
            const double u1 = (sm_red[2][0] + sm_red[2][1]) + (sm_red[2][2] + sm_red[2][3]);
            const double u2 = (sm_red[3][0] + sm_red[3][1]) + (sm_red[3][2] + sm_red[3][3]);
            const double ub = fmax(fmax(sm_red[4][0], sm_red[4][1]), fmax(sm_red[4][2], sm_red[4][3]));
            bool plain = ub < kComplementBelow * Hd;               // every mean width above 1/2
            for (int h = 0; h < H; ++h) plain = plain && sm_al[h] == 1.0 && sm_au[h] == 1.0;
            if (plain) {
                omega = Vd - (u1 + Vd * KC) / Hd;
                var = fmax(0.0, u2 - u1 * u1 / Vd) / (Hd * Hd * Vd);
            }
        }
        const double sigma = sqrt(var), score = omega * sigma;
        if (A.omega) A.omega[row] = (float)omega;
        if (A.sigma) A.sigma[row] = (float)sigma;
        if (A.score) A.score[row] = (float)score;
        if (A.flags) A.flags[row] = (uint8_t)(score > A.tau);
        if (A.p_lo || A.p_mid || A.p_hi) {
            int xid;
            if (A.ids) {
                xid = A.ids[row];
                xid = xid < 0 ? 0 : (xid >= V ? V - 1 : xid);
            } else {
                const float rm = fmaxf(fmaxf(sm_pm[0], sm_pm[1]), fmaxf(sm_pm[2], sm_pm[3]));
                xid = INT_MAX;
                for (int w = 0; w < 4; ++w) if (sm_pm[w] == rm && sm_pi[w] < xid) xid = sm_pi[w];
                if (xid == INT_MAX) xid = 0;
            }
            double lo = 0.0, mid = 0.0, hi = 0.0;
            for (int h = 0; h < H; ++h) {
                const T* crow = static_cast<const T*>(A.draft) + (int64_t)h * head_stride + row * A.stride;
                const double ex = (double)Elt<T>::exp2_ref(load_logit(crow, xid), sm_n[h]);
                const double x = ex / sm_S[h], omx = fmax(0.0, sm_S[h] - ex) / sm_S[h];
                double a = A.a, b = A.b;
                if (rad) {
                    const T* rrow = static_cast<const T*>(A.radius) + (int64_t)h * head_stride + row * A.stride;
                    const double r = radius_of((double)load_logit(rrow, xid), A.kappa, A.rmax);
                    a = exp(r); b = exp(-r);
                }
                mid += x;
                lo += sm_al[h] * b * x / (b + (1.0 - b) * omx);
                hi += sm_au[h] * a * x / (1.0 + (a - 1.0) * x);
            }
            if (A.p_lo) A.p_lo[row] = (float)(lo / Hd);
            if (A.p_mid) A.p_mid[row] = (float)(mid / Hd);
            if (A.p_hi) A.p_hi[row] = (float)(hi / Hd);
        }
    }
}

// Values that are the same in every lane of a wave, moved to scalar registers.
__device__ __forceinline__ double uniform_d(double v)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ FuseRow uniform_fr(FuseRow r)
{
    r.cu = uniform_f(r.cu); r.nih = uniform_f(r.nih); r.nil = uniform_f(r.nil); r.b = uniform_f(r.b); r.omb = uniform_f(r.omb);
    return r;
}
// 2^k as a double for an integer-valued float k of either sign (clamped to what leaves a sum finite)
__device__ __forceinline__ double pow2_any(float k) { return ldexp(1.0, (int)fminf(fmaxf(k, -1000.f), kFarUnits)); }

// Ensemble in one sweep, for up to kFusedHeads heads with a scalar radius whose rows fit a 512-lane workgroup
// (32 elements of a row per lane): every head's row of a position is read from memory once.  A workgroup takes one
// position at a time and two workgroups share a compute unit, one waiting for its rows while the other computes.
// The exponentials of two heads stay in registers; a third head's go through LDS (64 KiB per workgroup, each lane
// writing and reading its own slots), because three rows and the working set do not fit 128 registers.
// Per position:
//   1. as each head's row arrives: per-wave maximum, e_i = 2^(c_i log2e - n_w) in place of the logits, S_w;
//      -- barrier: the waves exchange (max, n_w, S_w) of every head --
//   2. every wave forms each head's S and reference.  Heads whose largest probability is below the host's bound
//      have inactive caps; if some head may have an active cap, every head's sums of p^l and of the widths are
//      taken first (one more exchange), which gives the caps.
//   3. D_i = sum_h delta_{h,i} token by token, sum (D_i - K), sum (D_i - K)^2 about the D of the position's first
//      token;  -- barrier --  thread 0 writes the position's outputs.
// Token arithmetic is fp32 throughout: calls whose flat rows need fp64 tokens (needs_flat_pass: wide intervals on
// nearly uniform rows) are not taken by this kernel, see ensemble_fused_fits.
constexpr int kFusedHeads = 3;
constexpr int kFusedThreads = 512;
constexpr int kFusedWaves = kFusedThreads / 64;

template <typename T, int NVEC, int H, bool ARGMAX>
__global__ __launch_bounds__(kFusedThreads) __attribute__((amdgpu_waves_per_eu(4)))
void ensemble_fused_kernel(const RowArgs A, const int64_t head_stride)
{
    using E = Elt<T>;
    constexpr int EPV = E::kPerVec, EPT = NVEC * EPV, NW = kFusedWaves;
    constexpr int RH = H < 3 ? H : 2;                              // heads whose exponentials stay in registers
    constexpr bool LH = H == 3;                                    // the third head's go through LDS
    extern __shared__ u32x4 sm_e2[];                               // LH: [EPT / 4][kFusedThreads]
    __shared__ float sm_ref[H][NW][2];                             // per head and wave: largest logit, reference n_w
    __shared__ double sm_S[H][NW];                                 // S_w in units of 2^-n_w
    __shared__ double sm_cap[H][NW][2];                            // sum gl, sum gw of a wave, in row units of e
    __shared__ double sm_red[2][NW];
    __shared__ double sm_Sh[H], sm_alh[H], sm_auh[H];              // per head, for the loops over a run-time h
    __shared__ float sm_nh[H];
    __shared__ float sm_pm[NW];
    __shared__ int sm_pi[NW];

    // (the wave's index lives in a scalar register and the lane's index is asked for again for every position: no
    // vector register is held for them)
    const int wave_s = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int V = A.V;
    const int nvec = (V + EPV - 1) / EPV;
    const bool partial = V < NVEC * kFusedThreads * EPV;           // the row does not fill the tile

    // Wave priority by progress, as in the streaming kernel: the two workgroups of a compute unit are served oldest
    // first; the one behind gets the higher priority, so that they end together.  (32-bit row arithmetic: scalar.)
    const uint32_t n_rows = (uint32_t)A.N, g_step = gridDim.x;
    const uint32_t my_cnt = blockIdx.x < n_rows ? (n_rows - blockIdx.x + g_step - 1u) / g_step : 0u;
    uint32_t done = 0;
    for (int64_t row = blockIdx.x; row < A.N; row += gridDim.x, ++done) {
        if (my_cnt > 1u) {
            if (done < ((my_cnt + 3u) >> 2)) __builtin_amdgcn_s_setprio(3);
            else if (done < ((my_cnt + 1u) >> 1)) __builtin_amdgcn_s_setprio(2);
            else if (done < ((3u * my_cnt + 3u) >> 2)) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        // (the lane's offsets are formed anew for every position: hoisted out of the loop they would occupy registers
        // for the whole kernel)
        // (likewise the radius constants: what is derived from them is cheap, and uniform)
        uint32_t ones = ~0u;
        double ra = A.a, rb = A.b;
        asm volatile("" : "+s"(ones), "+s"(ra), "+s"(rb));
        const int lane = (int)__builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0u));
        const int wave = wave_s, t = wave_s * 64 + lane;
        // one head's row of this position goes in flight (a scalar base address and a 32-bit lane offset)
        auto request = [&](u32x4 (&buf)[NVEC], int h) {
            const uint64_t b = (uint64_t)(static_cast<const T*>(A.draft) + (int64_t)h * head_stride + row * A.stride);
            const uint32_t blo = __builtin_amdgcn_readfirstlane((uint32_t)b);
            const uint32_t bhi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
            const gbytes base = (gbytes)(((uint64_t)bhi << 32) | blo);
            if (partial) {
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    const uint32_t off = (uint32_t)min(j * kFusedThreads + t, nvec - 1) * 16u;
                    buf[j] = __builtin_nontemporal_load((gvec)(base + off));
                }
            } else {
                const uint32_t off = (uint32_t)t * 16u;
#pragma unroll
                for (int j = 0; j < NVEC; ++j)
                    buf[j] = __builtin_nontemporal_load((gvec)(base + (uint64_t)j * (kFusedThreads * 16u) + off));
            }
        };
        // ---- 1: a head's row as it arrives: per-wave maximum, exponentials about the wave's integer reference, S_w
        auto stats = [&](u32x4 (&buf)[NVEC], float (&e)[EPT], int h, float& emax_w) -> float {
            if (partial) {
#pragma unroll
                for (int j = 0; j < NVEC; ++j) E::mask_tail(buf[j], (j * kFusedThreads + t) * EPV, V);
            }
#pragma unroll
            for (int j = 0; j < NVEC; ++j) E::unpack(buf[j], &e[j * EPV]);
            float ml = e[0];
#pragma unroll
            for (int i = 1; i < EPT; ++i) ml = fmaxf(ml, e[i]);
            const float mw = wave_max(ml);
            const float nw = ref_of(mw);
            const float nref = nw == -INFINITY ? 0.f : nw;
            double sacc = 0.0;                                     // (one accumulator: registers are scarcer here than issue slots)
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    e[j * EPV + k] = Elt<T>::exp2_ref(e[j * EPV + k], nref);
                    sacc += (double)e[j * EPV + k];
                }
                __builtin_amdgcn_sched_barrier(0);                 // keep the working set to one vector at a time
            }
            const double Sw = wave_sum(sacc);
            if (lane == 0) { sm_ref[h][wave][0] = mw; sm_ref[h][wave][1] = nw; sm_S[h][wave] = Sw; }
            emax_w = uniform_f(Elt<T>::exp2_ref(mw, nref));                // the wave's largest e_i, in its own units
            return uniform_f(nw);
        };
        float e[RH][EPT];
        float nwv[H], emw[H];
        if constexpr (LH) {
            // the third head first: its exponentials leave for LDS, and the second head's row is requested into
            // the registers that this frees
            u32x4 b0[NVEC];
            {
                u32x4 b2[NVEC];
                request(b2, 2);
                request(b0, 0);
                float e2[EPT];
                nwv[2] = stats(b2, e2, 2, emw[2]);
#pragma unroll
                for (int q = 0; q < EPT / 4; ++q) {
                    u32x4 w;
                    w.x = __float_as_uint(e2[q * 4]); w.y = __float_as_uint(e2[q * 4 + 1]);
                    w.z = __float_as_uint(e2[q * 4 + 2]); w.w = __float_as_uint(e2[q * 4 + 3]);
                    sm_e2[q * kFusedThreads + t] = w;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            nwv[0] = stats(b0, e[0], 0, emw[0]);
            __builtin_amdgcn_sched_barrier(0);
            u32x4 b1[NVEC];
            request(b1, 1);
            __builtin_amdgcn_sched_barrier(0);
            nwv[1] = stats(b1, e[1], 1, emw[1]);
        } else {
            u32x4 buf[RH][NVEC];
#pragma unroll
            for (int h = 0; h < RH; ++h) request(buf[h], h);
#pragma unroll
            for (int h = 0; h < RH; ++h) nwv[h] = stats(buf[h], e[h], h, emw[h]);
        }
        // element i of head h as this lane holds it
        auto e_of = [&](int h, int i, const u32x4& from_lds) -> float {
            if (h < RH) return e[h][i];
            const int c = i & 3;
            return __uint_as_float(c == 0 ? from_lds.x : c == 1 ? from_lds.y : c == 2 ? from_lds.z : from_lds.w);
        };
        __syncthreads();
        // ---- 2: every head's S and reference; which heads can have an active cap ---------------------------------
        double S[H];                                               // in units of 2^-n
        float n[H];
        bool all_capless = true, any_split = false;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            float mc = sm_ref[h][0][0], nn = sm_ref[h][0][1];
#pragma unroll
            for (int w = 1; w < NW; ++w) { mc = fmaxf(mc, sm_ref[h][w][0]); nn = fmaxf(nn, sm_ref[h][w][1]); }
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float rn = sm_ref[h][w][1];
                if (rn != -INFINITY) s += sm_S[h][w] * pow2_of(rn - nn);
            }
            S[h] = uniform_d(s); n[h] = uniform_f(nn);
            const double emax = (double)Elt<T>::exp2_ref(uniform_f(mc), n[h]);
            all_capless = all_capless && (!A.normalize || emax <= A.capless_xmax * S[h]);
            any_split = any_split || emax > 0.5 * S[h];
            __builtin_amdgcn_sched_barrier(0);                     // one head at a time: the LDS reads of all heads at once
                                                                   // would need registers that hold the rows
        }
        // this wave's units: its e_i are 2^(n - n_w) times the row's, and so is the partition sum it divides by
        double Sw_units[H];
#pragma unroll
        for (int h = 0; h < H; ++h)
            Sw_units[h] = nwv[h] != -INFINITY ? uniform_d(S[h] * pow2_any(n[h] - nwv[h])) : 1.0;
        double al[H], au[H];
#pragma unroll
        for (int h = 0; h < H; ++h) { al[h] = 1.0; au[h] = 1.0; }
        if (!all_capless) {                                        // uniform over the workgroup
            // sum p^l and sum of the widths of every head -> that head's caps
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const FuseRow fr = uniform_fr(fuse_row(Sw_units[h], ra, rb));
                double g0 = 0.0, g1 = 0.0;
#pragma unroll
                for (int q = 0; q < EPT / 4; ++q) {
                    u32x4 w = {0u, 0u, 0u, 0u};
                    if (h >= RH) w = sm_e2[q * kFusedThreads + t];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float gl, gw;
                        fuse_token(e_of(h, q * 4 + c, w), fr, gl, gw);
                        g0 += (double)gl; g1 += (double)gw;        // (a slot past the row's end holds e = 0: gl = gw = 0)
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // back to row units of e: a power of two
                const double fw = nwv[h] != -INFINITY ? pow2_of(nwv[h] - n[h]) : 0.0;
                g0 = wave_sum(g0) * fw; g1 = wave_sum(g1) * fw;
                if (lane == 0) { sm_cap[h][wave][0] = g0; sm_cap[h][wave][1] = g1; }
            }
            __syncthreads();
#pragma unroll
            for (int h = 0; h < H; ++h) {
                double sgl = 0.0, sgw = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) { sgl += sm_cap[h][w][0]; sgw += sm_cap[h][w][1]; }
                const double Sl = fmin(1.0, rb / S[h] * sgl), Su = fmax(1.0, rb / S[h] * sgl + (ra - rb) / S[h] * sgw);
                if (A.normalize) { al[h] = uniform_d(fmin(1.0, A.cap_lo / Sl)); au[h] = uniform_d(fmax(1.0, A.cap_hi / Su)); }
            }
        }
        if (t == 0) {
#pragma unroll
            for (int h = 0; h < H; ++h) { sm_Sh[h] = S[h]; sm_nh[h] = n[h]; sm_alh[h] = al[h]; sm_auh[h] = au[h]; }
        }
        // The sums over the tokens are taken about the D of the position's first token (every lane forms the same
        // number, from the logits in memory and the row's constants).
        double KD = 0.0;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const T* crow = static_cast<const T*>(A.draft) + (int64_t)h * head_stride + row * A.stride;
            const float e0 = Elt<T>::exp2_ref(load_logit(crow, 0), n[h]);
            float gl, gw;
            fuse_token(e0, fuse_row(S[h], ra, rb), gl, gw);
            KD = fma(au[h] * (ra - rb) / S[h], (double)gw, fma((au[h] - al[h]) * rb / S[h], (double)gl, KD));
        }
        KD = uniform_d(KD);
        double s1 = 0.0, s2 = 0.0;
        float best = -INFINITY;
        int best_i = INT_MAX;
        {
            // ---- 3: D_i in this wave's units of every head ---------------------------------------------------------
            FuseRow fr[H];
            double cw[H], cl[H];
            float invS[H];
#pragma unroll
            for (int h = 0; h < H; ++h) {
                fr[h] = uniform_fr(fuse_row(Sw_units[h], ra, rb));
                cw[h] = uniform_d(au[h] * (ra - rb) / Sw_units[h]);
                cl[h] = uniform_d((au[h] - al[h]) * rb / Sw_units[h]);
                invS[h] = uniform_f((float)(1.0 / Sw_units[h]));
            }
            // Specialised on what is uniform over the position or the wave: NOLOW = no head has an active cap (delta = w:
            // p^l is not needed), SPLIT = some probability above 1/2 (1 - x needs the two-float 1/S, see fuse_parts),
            // POLY = every token this wave holds, in every head, is small enough for the width polynomial that the host
            // has fitted for the call's radius (gw = e (1 + x P(x)), see RowArgs::wpoly): five FMAs instead of the
            // rational form with its reciprocal.
            float pd[H][4];
            bool poly = all_capless && A.wpoly_x >= 0.f;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const float is = -fr[h].nih, is2 = is * is;
                pd[h][0] = uniform_f(A.wpoly[0] * is); pd[h][1] = uniform_f(A.wpoly[1] * is2);
                pd[h][2] = uniform_f(A.wpoly[2] * (is2 * is)); pd[h][3] = uniform_f(A.wpoly[3] * (is2 * is2));
                poly = poly && ref_is_near(n[h]) && (double)emw[h] <= (double)A.wpoly_x * Sw_units[h];
            }
            auto sweep = [&](auto nolow_c, auto split_c, auto poly_c) {
                constexpr bool NOLOW = decltype(nolow_c)::value, SPLIT = decltype(split_c)::value;
                constexpr bool POLY = decltype(poly_c)::value;
#pragma unroll
                for (int q = 0; q < EPT / 4; ++q) {
                    const int j = q * 4 / EPV;
                    if (j * kFusedThreads * EPV >= V) continue;      // uniform: the chunk holds no token
                    u32x4 w = {0u, 0u, 0u, 0u};
                    if constexpr (LH) w = sm_e2[q * kFusedThreads + t];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int i = q * 4 + c;
                        double D = 0.0;
                        float pm = 0.f;
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            const float eh = e_of(h, i, w);
                            if constexpr (POLY) {
                                const float G = fmaf(fmaf(fmaf(fmaf(pd[h][3], eh, pd[h][2]), eh, pd[h][1]), eh, pd[h][0]), eh, 1.0f);
                                D = fma(cw[h], (double)(eh * G), D);
                            } else {
                                float g, du, om;
                                fuse_parts<SPLIT>(eh, fr[h], g, du, om);
                                D = fma(cw[h], (double)(g * om), D);
                                if constexpr (!NOLOW) D = fma(cl[h], (double)(g * du), D);
                            }
                            if (ARGMAX) pm = fmaf(eh, invS[h], pm);
                        }
                        // A slot past the row's end holds e = 0 in every head: D = 0 exactly, so it adds -KD and KD^2
                        // to the two sums, which thread 0 takes out again (the number of such slots is known); its mean
                        // probability 0 never wins the arg-max (strict comparison, and the lane's real tokens come first).
                        const double d = D - KD;
                        s1 += d;
                        s2 = fma(d, d, s2);
                        if (ARGMAX && pm > best) { best = pm; best_i = (j * kFusedThreads + t) * EPV + (i - j * EPV); }
                        if (c & 1) __builtin_amdgcn_sched_barrier(0);  // two tokens at a time: bounded working set
                    }
                }
            };
            using yes = std::integral_constant<bool, true>;
            using no = std::integral_constant<bool, false>;
            if (poly) sweep(yes{}, no{}, yes{});                    // (uniform over the wave)
            else if (all_capless) { if (any_split) sweep(yes{}, yes{}, no{}); else sweep(yes{}, no{}, no{}); }
            else { if (any_split) sweep(no{}, yes{}, no{}); else sweep(no{}, no{}, no{}); }
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if (lane == 0) { sm_red[0][wave] = s1; sm_red[1][wave] = s2; }
        if (ARGMAX) {
            // each lane walked its tokens in ascending order, so it holds its lowest index of its maximum
            const float wm = wave_max(best);
            const int wi = wave_min_i(best == wm ? best_i : INT_MAX);
            if (lane == 0) { sm_pm[wave] = wm; sm_pi[wave] = wi; }
        }
        __syncthreads();
        if (t == 0) {
            int Vr = V;
            asm volatile("" : "+s"(Vr));                           // (so that its conversion stays in this block)
            const double Hd = (double)H, Vd = (double)Vr;
            double t1 = 0.0, t2 = 0.0;
            for (int w = 0; w < NW; ++w) { t1 += sm_red[0][w]; t2 += sm_red[1][w]; }
            {
                // the slots of the tile past the row's end (chunks that hold no token at all were skipped)
                const int chunks = (Vr + kFusedThreads * EPV - 1) / (kFusedThreads * EPV);
                const double pad = (double)(chunks * kFusedThreads * EPV - Vr);
                t1 += pad * KD;
                t2 -= pad * KD * KD;
            }
            const double omega = (t1 + Vd * KD) / Hd;
            const double var = fmax(0.0, t2 - t1 * t1 / Vd) / (Hd * Hd * Vd);
            const double sigma = sqrt(var), score = omega * sigma;
            if (A.omega) A.omega[row] = (float)omega;
            if (A.sigma) A.sigma[row] = (float)sigma;
            if (A.score) A.score[row] = (float)score;
            if (A.flags) A.flags[row] = (uint8_t)(score > A.tau);
            if (A.p_lo || A.p_mid || A.p_hi) {
                int xid;
                if (A.ids) {
                    xid = A.ids[row];
                    xid = xid < 0 ? 0 : (xid >= V ? V - 1 : xid);
                } else {
                    float rm = sm_pm[0];
                    for (int w = 1; w < NW; ++w) rm = fmaxf(rm, sm_pm[w]);
                    xid = INT_MAX;
                    for (int w = 0; w < NW; ++w) if (sm_pm[w] == rm && sm_pi[w] < xid) xid = sm_pi[w];
                    if (xid == INT_MAX) xid = 0;
                }
                double lo = 0.0, mid = 0.0, hi = 0.0;
#pragma nounroll
                for (int h = 0; h < H; ++h) {
                    const T* crow = static_cast<const T*>(A.draft) + (int64_t)h * head_stride + row * A.stride;
                    const double Sh = sm_Sh[h];
                    const double ex = (double)Elt<T>::exp2_ref(load_logit(crow, xid), sm_nh[h]);
                    const double x = ex / Sh, omx = fmax(0.0, Sh - ex) / Sh;
                    mid += x;
                    lo += sm_alh[h] * rb * x / (rb + (1.0 - rb) * omx);
                    hi += sm_auh[h] * ra * x / (1.0 + (ra - 1.0) * x);
                }
                if (A.p_lo) A.p_lo[row] = (float)(lo / Hd);
                if (A.p_mid) A.p_mid[row] = (float)(mid / Hd);
                if (A.p_hi) A.p_hi[row] = (float)(hi / Hd);
            }
        }
        // (the next position's first barrier separates this read of sm_red / sm_pm from their next writes)
    }
}

// Ensemble in one sweep: every row of a position -- H centre rows and, with a radius tensor, H raw-radius rows -- is read
// from memory once.  A workgroup takes one position at a time and its heads one after another:
//   1. the head's centre row: per-wave maximum, e_i = 2^(c_i log2e - n_w), S_w;  -- barrier: (max, n_w, S_w) --
//   2. with S known, the head's widths, added to D_i = sum_h w_{h,i} token by token (fp64 registers), and where its caps
//      may be active the sums of p^l and of the widths.
// No row has to be kept for a later head: of a position only the D_i stay, so any number of heads fits the registers, and
// the next two rows are on their way into LDS all the time.  What binds is instructions: a row costs a wave ~350 of them
// whatever its length (reductions, the exchange, row constants), so a lane takes 32 tokens (e 32, D 64 registers) and two
// waves per SIMD share the registers; with 16 tokens per lane and four waves per SIMD the same call took 150-169 us
// (2048 x 16384 x 3 heads fp32 with radius; two sweeps over every row: 318 us).  Omega = sum D_i / H and Sigma^2 = sum D_i^2 / (H^2 V) - (Omega / V)^2 hold as they stand when no head has an active
// cap.  The positions where one has are swept a second time, with the caps known, when the workgroup is through with
// its positions.  Those whose D_i agree to better than a hundredth of their mean (fp64 sums about 0 lose nothing elsewhere),
// rows flat in every head and widths that all crowd against 1 are swept a second time in fp64.
// The positions' scalars are parked in LDS and turned into outputs after the workgroup's last one, a lane per position: the
// logits of the reported tokens are then fetched for all of them at once instead of in a chain per position.
constexpr int kSweepTokens = 32;                                   // tokens of a row per lane
template <int THREADS> constexpr int sweep_rows() { return THREADS >= 256 ? 32 : THREADS / 8; }   // most positions of a workgroup

// ARGMAX = no drafted ids: the reported token is the arg-max of the averaged centre distribution.
template <typename T, int THREADS, bool RAD, bool UNIT, bool ARGMAX>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2)))
void ensemble_sweep_kernel(const RowArgs A, const int H, const int64_t head_stride, const int wide,
                           const int flat_in_fp64)
{
    using E = Elt<T>;
    constexpr int EPV = E::kPerVec, NVEC = kSweepTokens / EPV, NW = THREADS / 64, ROWS = sweep_rows<THREADS>();
    extern __shared__ u32x4 sm_next[];                             // [2][NVEC][THREADS]: the two rows in flight
    // exchange slots: written before an item's barrier, read behind it; items (a head of a position) alternate between two
    __shared__ float sm_ref[2][NW][2];                             // per wave: largest logit, reference n_w
    __shared__ double sm_S[2][NW];
    __shared__ double sm_red[NW][48];                              // per wave: the slots of wave_sum3
    // a position's sums per wave, read by wave 0 behind the next position's first barrier; positions alternate
    __shared__ double sm_cap[2][kMaxHeads][2][NW];
    __shared__ double sm_sum[2][2][NW];
    __shared__ float sm_min[2][NW], sm_pm[2][NW];
    __shared__ int sm_pi[2][NW];
    // parked positions
    __shared__ double pk_S[ROWS][kMaxHeads], pk_al[ROWS][kMaxHeads], pk_au[ROWS][kMaxHeads];
    __shared__ double pk_sum[ROWS][2];
    __shared__ float pk_n[ROWS][kMaxHeads], pk_mc[ROWS][kMaxHeads];
    __shared__ int pk_id[ARGMAX ? ROWS : 1];
    __shared__ int pk_state[ROWS];                           // see kDone ...
    constexpr int kDone = 0, kCaps = 1, kFp64 = 2;                 // finished / an active cap / to be swept in fp64

    // (the lane's index is asked for anew wherever it is used, through an empty asm: no LDS address formed from it is
    // held in registers, or spilled, through the loop -- and a reload would wait for the rows in flight)
    auto my_tid = []() {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int V = A.V;
    const int last_vec = (V + EPV - 1) / EPV - 1;
    const bool partial = V < THREADS * kSweepTokens;               // the row does not fill the tile
    RadiusMode rm = {false, 0.f, 0.f, 0.f};
    if constexpr (RAD) {
        rm = radius_mode(A);
        rm.kappa = uniform_f(rm.kappa); rm.rmax = uniform_f(rm.rmax); rm.am1_max = uniform_f(rm.am1_max);
    }
    const uint32_t n_rows = (uint32_t)A.N, step = gridDim.x;

    using lds_ptr = __attribute__((address_space(3))) void*;
    using glb_ptr = const __attribute__((address_space(1))) void*;
    auto row_base = [&](const void* rows, uint32_t row, int h) {
        const uint64_t b = (uint64_t)(static_cast<const T*>(rows) + (int64_t)h * head_stride + (int64_t)row * A.stride);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
        return (gbytes)(((uint64_t)hi << 32) | lo);
    };
    // A row goes in flight, straight into LDS (lane l of a wave lands 16 l bytes behind the address the wave names; no
    // register is held while it is on its way).  A lane reads back only what its own wave has requested, so the
    // hand-over is the wave's own count of outstanding loads and no barrier.  whole = false: there is no such row; a few
    // bytes are fetched all the same, so that the count is the same.
    auto fetch = [&](int slot, const void* rows, uint32_t row, int h, bool whole, int tid) {
        const gbytes base = row_base(rows, row, h);
        if (partial || !whole) {
            const int t = whole ? tid : 0, end = whole ? last_vec : 0;
#pragma unroll
            for (int j = 0; j < NVEC; ++j)
                __builtin_amdgcn_global_load_lds((glb_ptr)(base + (uint32_t)min(j * THREADS + t, end) * 16u),
                                                 (lds_ptr)(sm_next + (slot * NVEC + j) * THREADS + wave * 64), 16, 0, kNonTemporal);
        } else {
            const uint32_t off = (uint32_t)tid * 16u;
#pragma unroll
            for (int j = 0; j < NVEC; ++j)
                __builtin_amdgcn_global_load_lds((glb_ptr)(base + (uint64_t)j * (THREADS * 16u) + off),
                                                 (lds_ptr)(sm_next + (slot * NVEC + j) * THREADS + wave * 64), 16, 0, kNonTemporal);
        }
    };
    // the older of the two rows in flight has landed; it moves to registers and its slot is free again
    auto take = [&](int slot, u32x4 (&buf)[NVEC], int tid) {
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NVEC) : "memory");
#pragma unroll
        for (int j = 0; j < NVEC; ++j) buf[j] = sm_next[(slot * NVEC + j) * THREADS + tid];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    // (the second sweep of a position: a row into registers)
    auto request = [&](u32x4 (&buf)[NVEC], const void* rows, uint32_t row, int h, int tid) {
        const gbytes base = row_base(rows, row, h);
#pragma unroll
        for (int j = 0; j < NVEC; ++j)
            buf[j] = __builtin_nontemporal_load((gvec)(base + (uint32_t)min(j * THREADS + tid, last_vec) * 16u));
    };
    auto unpack_row = [&](u32x4 (&buf)[NVEC], float (&v)[kSweepTokens], bool centre, int tid) {
        if (partial) {
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
                if (centre) E::mask_tail(buf[j], (j * THREADS + tid) * EPV, V);
                else E::zero_tail(buf[j], (j * THREADS + tid) * EPV, V);
            }
        }
#pragma unroll
        for (int j = 0; j < NVEC; ++j) E::unpack(buf[j], &v[j * EPV]);
    };
    auto sum_of_position = [&](const double (&D)[kSweepTokens], int p) {
        const int lane = my_tid() & 63;
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int i = 0; i < kSweepTokens; ++i) { s1 += D[i]; s2 = fma(D[i], D[i], s2); }
        s1 = wave_sum(s1); s2 = wave_sum(s2);
        if (lane == 0) { sm_sum[p][0][wave] = s1; sm_sum[p][1][wave] = s2; }
    };
    // wave 0: the sums of a position over the waves -> whether they are to be done again in fp64
    auto total_of_position = [&](int at, int p) {
        const int lane = my_tid() & 63;
        const int src = lane < NW ? lane : 0;
        const double s1 = row16_sum(lane < NW ? sm_sum[p][0][src] : 0.0), s2 = row16_sum(lane < NW ? sm_sum[p][1][src] : 0.0);
        // sum D_i and sum (D_i - mean)^2
        const double spread = s2 - s1 * s1 / (double)V;
        if (lane == 0) { pk_sum[at][0] = s1; pk_sum[at][1] = spread; }
        return !(spread >= 1e-4 * (s2 - spread));
    };
    // wave 0 parks a position: lane h settles head h's caps
    auto park = [&](int at, int p, bool all_flat, unsigned summed) {
        const int lane = my_tid() & 63;
        double al = 1.0, au = 1.0;
        if (lane < H) {
            if (A.normalize && (summed >> lane & 1u)) {
                double g0 = 0.0, g1 = 0.0;
                for (int w = 0; w < NW; ++w) { g0 += sm_cap[p][lane][0][w]; g1 += sm_cap[p][lane][1][w]; }
                al = fmin(1.0, A.cap_lo / fmin(1.0, g0));
                au = fmax(1.0, A.cap_hi / fmax(1.0, g0 + g1));
            }
            pk_al[at][lane] = al; pk_au[at][lane] = au;
        }
        const bool caps = __builtin_amdgcn_ballot_w64(al != 1.0 || au != 1.0) != 0;
        bool fp64 = total_of_position(at, p) || (all_flat && flat_in_fp64);
        if (wide) {
            // every mean width close to 1/2 or above it: the complements have to be looked at
            const int src = lane < NW ? lane : 0;
            const float least = -row16_max(lane < NW ? -sm_min[p][src] : -INFINITY);
            fp64 = fp64 || least > 0.45f * (float)H;
        }
        if constexpr (ARGMAX) {
            const float pm = lane < NW ? sm_pm[p][lane] : -INFINITY, top = row16_max(pm);
            const int best = wave_min_i(lane < NW && pm == top ? sm_pi[p][lane < NW ? lane : 0] : INT_MAX);
            if (lane == 0) pk_id[at] = best == INT_MAX ? 0 : best;
        }
        if (lane == 0) pk_state[at] = caps && !(all_flat && flat_in_fp64) ? kCaps : fp64 ? kFp64 : kDone;
    };

    uint32_t row = blockIdx.x;
    if (row >= n_rows) return;
    // With a radius tensor the two rows in flight are a head's centre row (slot 0) and its radius row (slot 1), each
    // requested when the one before it has moved to registers; without one, the centre rows of the next two heads.
    fetch(0, A.draft, row, 0, true, my_tid());
    if constexpr (RAD) fetch(1, A.radius, row, 0, true, my_tid());
    else fetch(1, A.draft, H > 1 ? row : row + step < n_rows ? row + step : row, H > 1 ? 1 : 0, true, my_tid());
    int done = 0, item = 0;
    bool flat_before = false;
    unsigned summed_before = 0;                                    // heads of the last position whose cap sums were taken
    for (;; ++done) {
        double D[kSweepTokens];
#pragma unroll
        for (int i = 0; i < kSweepTokens; ++i) D[i] = 0.0;
        float pm[ARGMAX ? kSweepTokens : 1];                       // the heads' probabilities added up
#pragma unroll
        for (int i = 0; i < (ARGMAX ? kSweepTokens : 1); ++i) pm[i] = 0.f;
        bool all_flat = true;
        unsigned summed = 0;
        const bool more_rows = row + step < n_rows && done + 1 < ROWS;
        for (int h = 0; h < H; ++h, ++item) {
            const int p = item & 1;
            const int tid = my_tid(), lane = tid & 63;
            // the item AHEAD items on (the same one where there is none)
            constexpr int AHEAD = RAD ? 1 : 2;
            uint32_t next_row = row;
            int next_h = h + AHEAD, next_done = done;
            while (next_h >= H) { next_h -= H; next_row += step; ++next_done; }
            const bool has_next = next_row < n_rows && next_done < ROWS;
            if (!has_next) { next_row = row; next_h = h; }
            // ---- 1: the centre row ---------------------------------------------------------------------------------
            float e[kSweepTokens];
            {
                u32x4 cbuf[NVEC];
                take(RAD ? 0 : p, cbuf, tid);
                fetch(RAD ? 0 : p, A.draft, next_row, next_h, has_next, tid);
                unpack_row(cbuf, e, true, tid);
            }
            const float mw = wave_max(max_of(e)), nw = ref_of(mw), nref = nw == -INFINITY ? 0.f : nw;
            double sacc[2] = {0.0, 0.0};
#pragma unroll
            for (int i = 0; i < kSweepTokens; ++i) {
                e[i] = Elt<T>::exp2_ref(e[i], nref);
                sacc[i & 1] += (double)e[i];
            }
            // S_w over the wave, together with the cap sums of the head before (in their slots since its end)
            double g0, g1, Sw = sacc[0] + sacc[1];
            wave_sum3_put(Sw, sm_red[wave], 2, lane);
            wave_sum3_get(sm_red[wave], lane, g0, g1, Sw);
            if (lane == 0) {
                sm_ref[p][wave][0] = mw; sm_ref[p][wave][1] = nw; sm_S[p][wave] = Sw;
                if (item > 0) {
                    const int hb = h > 0 ? h - 1 : H - 1, pb = h > 0 ? done & 1 : (done - 1) & 1;
                    sm_cap[pb][hb][0][wave] = g0; sm_cap[pb][hb][1][wave] = g1;
                }
            }
            lds_barrier();
            if (wave == 0 && h == 0 && done > 0) park(done - 1, (done - 1) & 1, flat_before, summed_before);
            // the waves' results combined, across the first lanes of every wave
            const int src = lane < NW ? lane : 0;
            // (the row's reference is the largest of the waves'; formed again from the largest logits, 600 x 3 x 1024 fp32 13.6 us
            // against 13.4)
            const float m_l = sm_ref[p][src][0], n_l = sm_ref[p][src][1], mc = row16_max(m_l), n = row16_max(n_l);
            const double S = row16_sum(lane < NW && n_l != -INFINITY ? sm_S[p][src] * pow2_of(n_l - n) : 0.0);
            // (the radius constants through an empty asm, formed anew for every row, and what is the same in every lane of
            // the wave moved to scalar registers: nothing of it is held in vector registers, or spilled, through the loop)
            double ra = A.a, rb = A.b;
            asm volatile("" : "+s"(ra), "+s"(rb));
            if (tid == 0) { pk_S[done][h] = S; pk_n[done][h] = n; pk_mc[done][h] = mc; }
            const double emax = (double)Elt<T>::exp2_ref(mc, n == -INFINITY ? 0.f : n);
            all_flat = all_flat && emax * (double)V <= 2.0 * S;
            const double Su = nw == -INFINITY ? 1.0 : ldexp(S, (int)fminf(n - nw, kFarUnits));   // S in this wave's units
            const double inv = uniform_d(recip(Su));
            // ---- 2: the head's widths ------------------------------------------------------------------------------
            const FuseRow fr = uniform_fr(fuse_row_inv(inv, ra, rb));
            const double cw = RAD ? inv : uniform_d((ra - rb) * inv);
            if constexpr (ARGMAX) {
                const float invf = (float)inv;
#pragma unroll
                for (int i = 0; i < kSweepTokens; ++i) pm[i] = fmaf(e[i], invf, pm[i]);
            }
            g0 = 0.0; g1 = 0.0;
            if constexpr (RAD) {
                float rv[kSweepTokens];
                {
                    u32x4 rbuf[NVEC];
                    take(1, rbuf, tid);
                    fetch(1, A.radius, next_row, next_h, has_next, tid);
                    unpack_row(rbuf, rv, false, tid);
                }
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    if (j * THREADS * EPV < V) {                   // uniform: the chunk holds tokens
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            float gl, gw;                          // (a slot past the row's end holds e = 0: both are 0)
                            fuse_token_rad<T, UNIT>(e[j * EPV + k], rv[j * EPV + k], fr, rm.kappa, rm.rmax, rm.am1_max, gl, gw);
                            const double w = (double)gw;
                            g0 += (double)gl; g1 += w;
                            D[j * EPV + k] = fma(cw, w, D[j * EPV + k]);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                g0 *= inv; g1 *= inv;
                summed |= 1u << h;
            } else {
                // (the host's bound on the largest probability, as in the streaming kernel)
                const bool capless = !A.normalize || emax <= A.capless_xmax * S;          // uniform over the workgroup
                const float is = -fr.nih, is2 = is * is;
                const bool poly = capless && A.wpoly_x >= 0.f && ref_is_near(n) && (double)Elt<T>::exp2_ref(mw, nref) <= (double)A.wpoly_x * Su;
                if (poly) {                                        // uniform over the wave: see RowArgs::wpoly
                    const float d0 = uniform_f(A.wpoly[0] * is), d1 = uniform_f(A.wpoly[1] * is2);
                    const float d2 = uniform_f(A.wpoly[2] * (is2 * is)), d3 = uniform_f(A.wpoly[3] * (is2 * is2));
#pragma unroll
                    for (int i = 0; i < kSweepTokens; ++i) {
                        const float G = fmaf(fmaf(fmaf(fmaf(d3, e[i], d2), e[i], d1), e[i], d0), e[i], 1.0f);
                        D[i] = fma(cw, (double)(e[i] * G), D[i]);
                        if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < kSweepTokens; ++i) {
                        float gl, gw;
                        fuse_token(e[i], fr, gl, gw);
                        const double w = (double)gw;
                        g0 += (double)gl; g1 += w;
                        D[i] = fma(cw, w, D[i]);
                        if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                    g0 *= rb * inv; g1 *= cw;
                }
                if (!capless) summed |= 1u << h;
            }
            wave_sum3_put(g0, sm_red[wave], 0, lane);
            wave_sum3_put(g1, sm_red[wave], 1, lane);
        }
        sum_of_position(D, done & 1);
        if constexpr (ARGMAX) {
            const int tid = my_tid();
            float best = -INFINITY;
            int at = INT_MAX;
#pragma unroll
            for (int i = 0; i < kSweepTokens; ++i) {               // (ascending tokens: the first of equal values stays)
                const int tok = (i / EPV * THREADS + tid) * EPV + i % EPV;
                if (tok < V && pm[i] > best) { best = pm[i]; at = tok; }
            }
            const float top = wave_max(best);
            at = wave_min_i(best == top ? at : INT_MAX);
            if ((tid & 63) == 0) { sm_pm[done & 1][wave] = top; sm_pi[done & 1][wave] = at; }
        }
        if (wide) {
            const int tid = my_tid();
            float least = INFINITY;
#pragma unroll
            for (int i = 0; i < kSweepTokens; ++i)
                if ((i / EPV * THREADS + tid) * EPV + i % EPV < V) least = fminf(least, (float)D[i]);
            least = -wave_max(-least);
            if ((tid & 63) == 0) sm_min[done & 1][wave] = least;
        }
        flat_before = all_flat;
        summed_before = summed;
        if (!more_rows) break;
        row += step;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // (the requests without a row have landed)
    {
        double g0, g1, g2;
        const int lane = my_tid() & 63;
        wave_sum3_get(sm_red[wave], lane, g0, g1, g2);
        if (lane == 0) { sm_cap[done & 1][H - 1][0][wave] = g0; sm_cap[done & 1][H - 1][1][wave] = g1; }
    }
    __syncthreads();
    if (wave == 0) park(done, done & 1, flat_before, summed_before);
    __syncthreads();
    // ---- the positions with an active cap once more: delta_i = alpha_u w_i + (alpha_u - alpha_l) p^l_i -----------------
    for (int at = 0; at <= done; ++at) {
        if (pk_state[at] != kCaps) continue;                       // uniform
        const uint32_t r = blockIdx.x + (uint32_t)at * step;
        const int tid = my_tid();
        double D[kSweepTokens];
#pragma unroll
        for (int i = 0; i < kSweepTokens; ++i) D[i] = 0.0;
        for (int h = 0; h < H; ++h) {
            u32x4 cbuf[NVEC], rbuf[NVEC];
            request(cbuf, A.draft, r, h, tid);
            if constexpr (RAD) request(rbuf, A.radius, r, h, tid);
            const double S = pk_S[at][h], al = pk_al[at][h], au = pk_au[at][h], inv = 1.0 / S;
            const float n = pk_n[at][h];
            const FuseRow fr = fuse_row(S, A.a, A.b);
            const double cw = au * (RAD ? inv : (A.a - A.b) * inv), cl = (au - al) * (RAD ? inv : A.b * inv);
            float e[kSweepTokens], rv[kSweepTokens];
            unpack_row(cbuf, e, true, tid);
            if constexpr (RAD) unpack_row(rbuf, rv, false, tid);
#pragma unroll
            for (int i = 0; i < kSweepTokens; ++i) {
                const float ek = Elt<T>::exp2_ref(e[i], n == -INFINITY ? 0.f : n);
                float gl, gw;
                if constexpr (RAD) fuse_token_rad<T, UNIT>(ek, rv[i], fr, rm.kappa, rm.rmax, rm.am1_max, gl, gw);
                else fuse_token(ek, fr, gl, gw);
                D[i] = fma(cw, (double)gw, fma(cl, (double)gl, D[i]));
                if ((i & 1) == 1) __builtin_amdgcn_sched_barrier(0);
            }
        }
        sum_of_position(D, 0);
        __syncthreads();
        if (wave == 0) {
            const bool fp64 = total_of_position(at, 0);
            if (my_tid() == 0) pk_state[at] = fp64 ? kFp64 : kDone;
        }
        __syncthreads();
    }
    // ---- and those that want fp64, from the logits; the sums about D and C of the position's first token, so that a spread
    // far below the mean is not the difference of two large moments.  C_i = sum_h (1 - width_{h,i}): where every mean width is
    // above 1/2 and no cap is active (wide calls), Omega and Sigma are taken from the C_i, which resolve a spread that the
    // widths, all rounding to 1, no longer show.
    for (int at = 0; at <= done; ++at) {
        if (pk_state[at] != kFp64) continue;                       // uniform
        const int64_t r = (int64_t)blockIdx.x + (int64_t)at * step;
        const int tid = my_tid();
        auto token = [&](int i, double& d, double& c) {
            d = 0.0; c = 0.0;
            for (int h = 0; h < H; ++h) {
                const int64_t off = (int64_t)h * head_stride + r * A.stride;
                const double S = pk_S[at][h];
                const double ed = exp(ln_exp2<T>(load_logit(static_cast<const T*>(A.draft) + off, i), (double)pk_n[at][h]));
                const double inv = recip(S), x = ed * inv, omx = fmax(0.0, S - ed) * inv;
                double a = A.a, b = A.b;
                if constexpr (RAD) {
                    const double rr = radius_of((double)load_logit(static_cast<const T*>(A.radius) + off, i), A.kappa, A.rmax);
                    a = exp(rr); b = exp(-rr);
                }
                const double du = 1.0 + (a - 1.0) * x, dl = b + (1.0 - b) * omx;
                d += pk_au[at][h] * a * x / du - pk_al[at][h] * b * x / dl;
                c += (1.0 - 2.0 * (1.0 - b) * x * omx) / (du * dl);
            }
        };
        double KD, KC;
        token(0, KD, KC);
        double q[4] = {0.0, 0.0, 0.0, 0.0}, most = 0.0;
        for (int i = tid; i < V; i += THREADS) {
            double d, c;
            token(i, d, c);
            most = fmax(most, c);
            d -= KD; c -= KC;
            q[0] += d; q[1] = fma(d, d, q[1]); q[2] += c; q[3] = fma(c, c, q[3]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            q[i] = wave_sum(q[i]);
            if ((tid & 63) == 0) sm_red[wave][i] = q[i];
        }
        most = wave_max(most);
        if ((tid & 63) == 0) sm_red[wave][4] = most;
        __syncthreads();
        if (tid == 0) {
            double t[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
            for (int w = 0; w < NW; ++w) {
                for (int i = 0; i < 4; ++i) t[i] += sm_red[w][i];
                t[4] = fmax(t[4], sm_red[w][4]);
            }
            bool plain = wide && t[4] < kComplementBelow * (double)H;
            for (int h = 0; h < H; ++h) plain = plain && pk_al[at][h] == 1.0 && pk_au[at][h] == 1.0;
            const double Vd = (double)V;
            pk_sum[at][0] = plain ? (double)H * Vd - (t[2] + Vd * KC) : t[0] + Vd * KD;
            pk_sum[at][1] = plain ? t[3] - t[2] * t[2] / Vd : t[1] - t[0] * t[0] / Vd;
        }
        __syncthreads();
    }
    // ---- a lane per position --------------------------------------------------------------------------------------
    const int t = my_tid();
    if (t > done) return;
    const int64_t r = (int64_t)blockIdx.x + (int64_t)t * step;
    const double Hd = (double)H, Vd = (double)V;
    const double omega = pk_sum[t][0] / Hd, sigma = sqrt(fmax(0.0, pk_sum[t][1]) / (Hd * Hd * Vd)), score = omega * sigma;
    if (A.omega) A.omega[r] = (float)omega;
    if (A.sigma) A.sigma[r] = (float)sigma;
    if (A.score) A.score[r] = (float)score;
    if (A.flags) A.flags[r] = (uint8_t)(score > A.tau);
    if (A.p_lo || A.p_mid || A.p_hi) {
        int xid = ARGMAX ? pk_id[ARGMAX ? t : 0] : A.ids[r];
        xid = xid < 0 ? 0 : (xid >= V ? V - 1 : xid);
        double lo = 0.0, mid = 0.0, hi = 0.0;
        for (int h = 0; h < H; ++h) {
            const T* crow = static_cast<const T*>(A.draft) + (int64_t)h * head_stride + r * A.stride;
            const double Sh = pk_S[t][h], ex = (double)Elt<T>::exp2_ref(load_logit(crow, xid), pk_n[t][h]);
            const double x = ex / Sh, omx = fmax(0.0, Sh - ex) / Sh;
            double a = A.a, b = A.b;
            if constexpr (RAD) {
                const T* rrow = static_cast<const T*>(A.radius) + (int64_t)h * head_stride + r * A.stride;
                const double rr = radius_of((double)load_logit(rrow, xid), A.kappa, A.rmax);
                a = exp(rr); b = exp(-rr);
            }
            mid += x;
            lo += pk_al[t][h] * b * x / (b + (1.0 - b) * omx);
            hi += pk_au[t][h] * a * x / (1.0 + (a - 1.0) * x);
        }
        if (A.p_lo) A.p_lo[r] = (float)(lo / Hd);
        if (A.p_mid) A.p_mid[r] = (float)(mid / Hd);
        if (A.p_hi) A.p_hi[r] = (float)(hi / Hd);
    }
}

// Voting: flags[row] = strict majority of head_flags[h][row].
__global__ __launch_bounds__(256) void vote_kernel(const uint8_t* __restrict__ head_flags, int H, int64_t N,
                                                   uint8_t* __restrict__ flags)
{
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= N) return;
    int votes = 0;
    for (int h = 0; h < H; ++h) votes += head_flags[(int64_t)h * N + row] != 0;
    flags[row] = (uint8_t)(2 * votes > H);
}

}  // namespace

int max_heads() { return kMaxHeads; }

hipError_t launch_ensemble(int dtype, const RowArgs& args, int heads, int64_t head_stride, hipStream_t stream)
{
    if (args.N <= 0) return hipSuccess;
    const dim3 grid((unsigned)args.N), block(256);
    if (wide_radius(args)) {
        if (dtype == 0) hipLaunchKernelGGL((ensemble_kernel<float, true>), grid, block, 0, stream, args, heads, head_stride);
        else hipLaunchKernelGGL((ensemble_kernel<bf16_t, true>), grid, block, 0, stream, args, heads, head_stride);
    } else {
        if (dtype == 0) hipLaunchKernelGGL((ensemble_kernel<float, false>), grid, block, 0, stream, args, heads, head_stride);
        else hipLaunchKernelGGL((ensemble_kernel<bf16_t, false>), grid, block, 0, stream, args, heads, head_stride);
    }
    return hipGetLastError();
}

// 32 tokens of a row per lane of at most 512: V <= 16384.  (The fp64 token path of tiny vocabularies is ensemble_kernel's.)
// Except for many heads of few, short rows: a position's heads take their turn in its workgroup, ~3 us each however short the
// row, and the two-sweep route has every head's row in a workgroup of its own first.  (8 positions, one sweep / two, scalar
// radius fp32: 8 heads of 1024 tokens 25.9 / 15.8 us, of 4096 23.9 / 21.7, of 8192 23.9 / 30.3; 5 heads of 1024 17.6 / 13.3, of
// 2048 16.1 / 13.9, of 4096 16.4 / 17.4.  Radius tensors: 34.4 / 25.5, 35.3 / 33.5; 23.3 / 20.8, 23.6 / 22.2, 24.0 / 26.4.  256
// positions of 4 heads of 1024 tokens 15.3 / 14.3 and 27.1 / 20.5, of 2048 13.9 / 15.1; 1000 of 5 heads of 1024 26.5 / 27.3.)
bool ensemble_sweep_fits(const RowArgs& args, int heads)
{
    if (args.V <= kTinyVocab || args.V > 512 * kSweepTokens) return false;
    return !(args.N <= compute_units() && 1024 * (heads - 3) >= args.V);
}

namespace {
template <typename T, int THREADS, bool RAD, bool UNIT, bool ARGMAX>
hipError_t launch_sweep_cfg(const RowArgs& a, int heads, int64_t head_stride, hipStream_t stream)
{
    constexpr unsigned lds = 2u * kSweepTokens * sizeof(T) * THREADS;              // two rows: 8 to 128 KiB
    {
        // with the static arrays above the default limit: raised once per device and instance
        static std::mutex guard;
        static bool raised[64] = {};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        std::lock_guard<std::mutex> lock(guard);
        if (!raised[dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&ensemble_sweep_kernel<T, THREADS, RAD, UNIT, ARGMAX>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            raised[dev] = true;
        }
    }
    const int64_t g = whole_rounds(a.N, sweep_rows<THREADS>(), (int64_t)(512 / THREADS) * compute_units());
    const int wide = wide_radius(a) ? 1 : 0, flat64 = a.radius || needs_flat_pass(a) ? 1 : 0;
    hipLaunchKernelGGL((ensemble_sweep_kernel<T, THREADS, RAD, UNIT, ARGMAX>), dim3((unsigned)g), dim3(THREADS), lds, stream, a, heads,
                       head_stride, wide, flat64);
    return hipGetLastError();
}
template <typename T, int THREADS, bool ARGMAX>
hipError_t launch_sweep_radius(const RowArgs& a, int heads, int64_t head_stride, hipStream_t stream)
{
    if (!a.radius) return launch_sweep_cfg<T, THREADS, false, false, ARGMAX>(a, heads, head_stride, stream);
    if (a.kappa == 1.0) return launch_sweep_cfg<T, THREADS, true, true, ARGMAX>(a, heads, head_stride, stream);
    return launch_sweep_cfg<T, THREADS, true, false, ARGMAX>(a, heads, head_stride, stream);
}
template <typename T, int THREADS>
hipError_t launch_sweep_tile(const RowArgs& a, int heads, int64_t head_stride, hipStream_t stream)
{
    const bool argmax = a.ids == nullptr && (a.p_lo || a.p_mid || a.p_hi);
    return argmax ? launch_sweep_radius<T, THREADS, true>(a, heads, head_stride, stream)
                  : launch_sweep_radius<T, THREADS, false>(a, heads, head_stride, stream);
}
template <typename T>
hipError_t launch_sweep_typed(const RowArgs& a, int heads, int64_t head_stride, hipStream_t stream)
{
    if (a.V <= 64 * kSweepTokens) return launch_sweep_tile<T, 64>(a, heads, head_stride, stream);
    if (a.V <= 128 * kSweepTokens) return launch_sweep_tile<T, 128>(a, heads, head_stride, stream);
    if (a.V <= 256 * kSweepTokens) return launch_sweep_tile<T, 256>(a, heads, head_stride, stream);
    return launch_sweep_tile<T, 512>(a, heads, head_stride, stream);
}
}  // namespace

hipError_t launch_ensemble_sweep(int dtype, const RowArgs& args, int heads, int64_t head_stride, hipStream_t stream)
{
    if (args.N <= 0) return hipSuccess;
    if (!ensemble_sweep_fits(args, heads)) return hipErrorInvalidValue;
    return dtype == 0 ? launch_sweep_typed<float>(args, heads, head_stride, stream)
                      : launch_sweep_typed<bf16_t>(args, heads, head_stride, stream);
}

// Where its four waves per SIMD beat ensemble_sweep_kernel's two: a lane's share of a row filled with 17 to 32 tokens
// (2048 positions x 16384 tokens, bf16: 58.8 against 68.2 us with two heads, 83.9 against 96.9 with three; fp32: 73.4 / 78.5,
// 98.1 / 100.2; with 8192 tokens x 4096 positions the other way round: bf16 80.2 against 72.6, 117 against 103; fp32 87.8 / 75.5,
// 127 / 107) -- and where there is a position per compute unit at most, whose heads it takes side by side (8 positions of 3
// heads of 1024 tokens 9.1 against 12.0, bf16 10.3 / 11.7, of 4096 9.7 / 11.3; 256 of 2 heads of 4096 tokens 7.5 / 9.1; 600 of 3 heads
// of 4096 20.0 / 17.0).
bool ensemble_fused_fits(const RowArgs& args, int heads)
{
    return !args.radius && !wide_radius(args) && !needs_flat_pass(args) && heads >= 1 && heads <= kFusedHeads && args.V > kTinyVocab &&
           args.V <= 32 * kFusedThreads && (args.V > 16 * kFusedThreads || args.N <= compute_units());
}

namespace {
template <typename T, int NVEC, int H>
hipError_t launch_ensemble_fused_heads(const RowArgs& a, int64_t head_stride, hipStream_t stream)
{
    const int64_t resident = 2 * (int64_t)compute_units();
    const dim3 grid((unsigned)(a.N < resident ? a.N : resident)), block(kFusedThreads);
    const bool argmax = a.ids == nullptr && (a.p_lo || a.p_mid || a.p_hi);
    // the third head's exponentials: 4 bytes x elements per lane x lanes (64 KiB for the largest tile), above the
    // default limit on dynamic LDS together with the static arrays: raised once per device and instance
    constexpr unsigned lds = H == 3 ? NVEC * Elt<T>::kPerVec * kFusedThreads * 4u : 0u;
    if (lds) {
        static std::mutex guard;
        static bool raised[2][64] = {};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        std::lock_guard<std::mutex> lock(guard);
        if (!raised[argmax ? 1 : 0][dev]) {
            const hipError_t e = argmax
                ? hipFuncSetAttribute(reinterpret_cast<const void*>(&ensemble_fused_kernel<T, NVEC, H, true>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)
                : hipFuncSetAttribute(reinterpret_cast<const void*>(&ensemble_fused_kernel<T, NVEC, H, false>),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            raised[argmax ? 1 : 0][dev] = true;
        }
    }
    if (argmax) hipLaunchKernelGGL((ensemble_fused_kernel<T, NVEC, H, true>), grid, block, lds, stream, a, head_stride);
    else hipLaunchKernelGGL((ensemble_fused_kernel<T, NVEC, H, false>), grid, block, lds, stream, a, head_stride);
    return hipGetLastError();
}
template <typename T, int NVEC>
hipError_t launch_ensemble_fused_cfg(const RowArgs& a, int heads, int64_t head_stride, hipStream_t stream)
{
    static_assert(kFusedHeads == 3, "one instance per number of heads");
    if (heads == 1) return launch_ensemble_fused_heads<T, NVEC, 1>(a, head_stride, stream);
    if (heads == 2) return launch_ensemble_fused_heads<T, NVEC, 2>(a, head_stride, stream);
    return launch_ensemble_fused_heads<T, NVEC, 3>(a, head_stride, stream);
}
}  // namespace

hipError_t launch_ensemble_fused(int dtype, const RowArgs& args, int heads, int64_t head_stride, hipStream_t stream)
{
    if (args.N <= 0) return hipSuccess;
    if (!ensemble_fused_fits(args, heads)) return hipErrorInvalidValue;
    const int epv = dtype == 0 ? 4 : 8, vecs = (args.V + epv - 1) / epv;
    const int per_lane = (vecs + kFusedThreads - 1) / kFusedThreads;
    if (dtype == 0) {
        if (per_lane <= 2) return launch_ensemble_fused_cfg<float, 2>(args, heads, head_stride, stream);
        if (per_lane <= 4) return launch_ensemble_fused_cfg<float, 4>(args, heads, head_stride, stream);
        return launch_ensemble_fused_cfg<float, 8>(args, heads, head_stride, stream);
    }
    if (per_lane <= 2) return launch_ensemble_fused_cfg<bf16_t, 2>(args, heads, head_stride, stream);
    return launch_ensemble_fused_cfg<bf16_t, 4>(args, heads, head_stride, stream);
}

hipError_t launch_vote(const uint8_t* head_flags, int heads, int64_t N, uint8_t* flags, hipStream_t stream)
{
    if (N <= 0) return hipSuccess;
    hipLaunchKernelGGL(vote_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, stream, head_flags, heads, N, flags);
    return hipGetLastError();
}

}  // namespace ciar
