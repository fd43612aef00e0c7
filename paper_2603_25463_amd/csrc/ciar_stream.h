// gfx950 streaming kernel of the CIAR quantify + verify pass (this file: the kernel and its launch; ciar_stream.hip, ciar_rows.hip and
// ciar_short.hip: its instances and which call takes which), with an overview of the pass.
//
//   stream_kernel   reads every logit row exactly once from HBM.  A workgroup of 256 lanes (512 or 1024 for large
//                   vocabularies or few rows) owns one row at a time and walks over rows blockIdx.x, blockIdx.x +
//                   gridDim.x, ...  The grid is the workgroups that are resident at once (four waves per SIMD;
//                   more, taking their turn, when a workgroup would otherwise get more than kMaxRowsPerWg rows):
//                   while one workgroup waits for its row, the others compute, which keeps the memory system busy
//                   without a second set of row registers.  Loads are interleaved over the workgroup so that every
//                   load instruction of a wave covers 1 KiB of consecutive memory, and non-temporal (every logit is
//                   used once).  Nothing V-wide is ever written back.
//                   What a row leaves behind (its statistics, the accept verdict, the draw of a rejected row) is
//                   parked in LDS, and after its last row the workgroup turns that into the rows' outputs, two
//                   lanes per row in fp64 (finish_batch): caps, Omega, Sigma, U, flag, the interval of the reported
//                   token, the exact accept test, the window outputs.  A call whose rows fit this scheme is this
//                   one launch.
//   resample_kernel (ciar_finish.hip) draws for the rejected rows of launches whose tiles cannot keep both rows in
//                   registers (wide radii, bf16 rows above 8192 tokens with a radius tensor), re-reading the two rows.
//
// The centre row has to be resident between its statistics pass and its interval pass: the InterFuse
// bounds need the partition sum S of the complete row before the first bound can be formed (App.
// "Proof of Interval Validity": S appears in every denominator).  It lives in registers as
// e_i = 2^(c_i log2e - n_w).  The verifier row is only needed for max / Z and is consumed on arrival.
//
// stream_kernel, per row (centre row first: it carries most of the arithmetic, so that little is left
// to do when the last bytes of a launch arrive):
//   B  centre row:   per-wave maximum, e_i = 2^(c_i log2e - n_w) kept in registers, S_w = sum e_i
//      The reference n_w is an integer (the next integer above max * log2e of the *wave*), so the
//      waves need no barrier before exponentiating and their results combine exactly:
//      S = sum_w S_w 2^(n_w - n), n = max_w n_w, a power-of-two rescale.
//   -- barrier: the waves exchange (max, n_w, S_w) --
//   C  InterFuse for a scalar radius r, a = e^r, b = e^-r, x_i = e_i / S:
//        p^u_i = a x_i / (1 + (a-1) x_i),   p^l_i = b x_i / (1 - (1-b) x_i)
//      with one reciprocal of the product of the two denominators, accumulated as the lower
//      bound p^l_i and the raw width w_i = p^u_i - p^l_i = (a-b) x_i (1-x_i) / (du_i dl_i):
//      five fp64 sums per row (sum p^l, sum w and the three second moments); two of them when the
//      row's largest probability shows that the caps cannot be active.
//   T  verifier row, loaded into the registers the centre row came in (requested before C where the
//      registers allow, else after it): per-wave maximum, Z_w = sum 2^(t_i log2e - nt_w)   (max-trick)
//   -- barrier: the waves exchange their interval sums and (nt_w, Z_w); thread 0 writes RowStats --
//
// finishing lanes / residual draw, per row (Eq. uncertainty_score; Algorithm 1's threshold and verification steps):
//   delta_i = alpha_u w_i + (alpha_u - alpha_l) p^l_i once the 0.99 / 1.01 caps alpha_l, alpha_u are
//   known, so Omega = sum delta_i, Sigma^2 = (sum delta_i^2) / V - (Omega / V)^2, U = Omega * Sigma
//   follow from the five sums without a second sweep over the row; flag = U > tau;
//   accept iff ln u < min(0, ln q_x - ln p_x) (log domain, fp64);
//   rejected rows: res_i = max(0, q_i - p_i), inverse-CDF draw in token order from a workgroup-wide
//   prefix sum.
//
// Sums over a row are accumulated per lane (S and the five interval sums in fp64, which this chip
// issues at the fp32 rate) and combined across lanes with DPP and across waves through LDS in a fixed
// order, so results are deterministic and the per-row scalars carry ~1e-8 relative error.
#pragma once

#include "ciar_device.h"
#include <hip/hip_ext.h>
#include <mutex>
#include <type_traits>

namespace ciar {

// A launch request: with `launch` unset the dispatch below only reports the grid it would use.
struct StreamLaunch {
    bool launch;
    bool finish_rows;      // the caller wants the kernel to finish its rows (launches with a verifier row always do)
    hipStream_t stream;
    int units;             // compute units of the device
    StreamPlan plan;       // out
    hipEvent_t ev_start, ev_stop;   // both or neither: recorded by the dispatch at the kernel's start and end
};

// Calls on bf16 rows of more than 8192 tokens with a verifier row, without a radius tensor and without complements (wide_radius).
hipError_t launch_both_rows(Mode mode, const RowArgs& a, StreamLaunch& s);
// Calls without a radius tensor and without complements, whose rows the kernel finishes, on short rows where there are enough of them.
bool short_rows_fit(Mode mode, int dtype, const RowArgs& a, int units);
hipError_t launch_short_rows(int dtype, Mode mode, const RowArgs& a, StreamLaunch& s);

namespace {

// ---- the streaming kernel ---------------------------------------------------------------------------------

// Waves per SIMD the register allocation aims for: the centre row held as floats plus ~40 working
// registers, capped at 4 waves.  Memory latency is hidden by the other resident workgroups of the compute
// unit rather than by fetching ahead into a second set of registers: measured on this chip, three or
// four resident workgroups beat two with a register prefetch of the next row at every vocabulary size.
// (Tensor-radius mode: the raw radius row sits in registers next to the centre row during the interval pass.)
// Short rows, many of them: a wave to a row, or two, of at most eight vectors per lane.  With 256 lanes to
// every row a row of 1024 tokens left a lane four of them, and the 415 instructions that a wave spends per row were nearly all of
// its work; here one wave has them all, no wave waits for another, and its rows come through LDS as below (16384 x 1024 fused bf16
// 90 -> 33 us, fp32 65 -> 35, quantified 50 -> 20 and 42 -> 21; the rule and more figures: short_rows_fit).
//
// Large bf16 rows with a verifier row: twelve or sixteen vectors per lane at two waves per SIMD, the rows arriving through LDS.
// Bound by vector instructions: 16.9 of them per position and token are the tokens' own arithmetic, what a wave does per row besides
// (reductions, exchange, accept test) is spread over 128 tokens of a lane instead of 64, and with 256 registers the exponentials
// of the centre row (128) and the packed verifier row (64) are both there when the accept test has been decided, so that the
// draws of rejected rows are made here and resample_kernel's second read of their rows (57 of 250 us, below) is gone.  (What does not fit
// 256 registers with sixteen vectors, 48 to 88 B per lane, lies in blocks away from the usual path, mostly of waves whose rows may not go through
// the matrix cores; twelve vectors fit.)
// Two waves hide less of each other's waiting than four, so the rows are requested by global_load_lds into one row of LDS per
// workgroup that takes them in turn -- the verifier row while the centre row is exponentiated, the next centre row during the
// rest -- and there is one barrier per row: the verifier row is summed ahead of the exchange, and the interval sums are handed
// over with the next row's.  (Twelve vectors: rows that would fill less than three quarters of sixteen.)
// us per call, tiles of eight vectors and resample_kernel / these: fused 16384 x 16384 260 / 243, 32768 x 65536 1900 / 1769 (on another card
// 235 and 1705), 2048 x 20000 78 / 64, 256 x 16384 24 / 19; verified 4099 x 32003 131 / 106, 520 x 9714 27 / 18, 64 x 40000 31 / 18.  Vector
// instructions busy 85 % of the time; a fused pass over rows that stay in the caches takes 186 us without its draws, 229 with.
// (Same tiles, fp32: 2048 x 16384 50 / 55; those calls wait for memory.  Voting with radius tensors, radius_lean_kernel with
// sixteen vectors: 106 / 121.)
template <typename T, int THREADS, int NVEC, bool DO_V, bool RAD, bool WIDE>
constexpr bool next_by_lds()
{
    return !RAD && !WIDE && (THREADS <= 64 || (DO_V && (NVEC == 16 || NVEC == 12)) || (THREADS == 128 && NVEC == 8));
}
// The first vectors of every lane that all rows of an instance fill: large bf16 rows, which take the tile of fewer vectors otherwise
// (launch_both_rows; launch_stream_kernel refuses others).
template <typename T, int THREADS, int NVEC, bool DO_V, bool RAD, bool WIDE>
constexpr int full_vectors()
{
    return next_by_lds<T, THREADS, NVEC, DO_V, RAD, WIDE>() && NVEC == 16 ? 12 : 0;
}
template <typename T, int THREADS, int NVEC, bool RAD, bool DO_V = false>
constexpr int target_waves()
{
    if (next_by_lds<T, THREADS, NVEC, DO_V, RAD, false>()) {
        constexpr int regs = NVEC * Elt<T>::kPerVec + (DO_V ? NVEC * 4 : 0) + 56;   // the centre row's exponentials, the verifier row, working registers
        return regs <= 128 ? 4 : regs <= 168 ? 3 : 2;
    }
    constexpr int ept = NVEC * Elt<T>::kPerVec;                    // one row as floats
    constexpr int fit = 512 / (ept + (RAD ? NVEC * 4 + 8 : 0) + 40);
    constexpr int lo = (THREADS + 255) / 256;                      // waves per SIMD one workgroup needs
    return fit < lo ? lo : (fit > 4 ? 4 : fit);
}

// The interval sums of a flat row are taken about a shift (kl, kw, kc): sum (gl - kl), sum (gw - kw) and their
// second moments.  A row of nearly equal logits has a spread far below its mean width: about the origin the
// difference of the second moment and the squared mean leaves rounding noise of relative size 1e-8 in Sigma,
// which Omega ~ V multiplies; about a point among the data it loses next to nothing.  "Flat" = the largest
// probability is at most 2 / V.  Elsewhere the spread is at least ~1 / sqrt(V) of the mean and plain sums do; a
// shift would even hurt there, because a token far below it keeps only ulp(k) / 2 of absolute accuracy in gl - k,
// which over a row of small tokens adds up to V * 3e-8 * k.
// Scalar radius: the shift is the token function at the mean of the row's e_i, S / V.  Tensor radius: the values
// of the row's first token.  Every wave forms the shift itself in its own units, a power of two away from the
// others', so the shifts agree bit for bit once they are back in row units and the waves' sums simply add.
struct Shift { float kl, kw, kc; };

// Pass C for one lane: the shifted InterFuse sums over the lane's tokens.  gl - kl and gw - kw come out of the
// FMA that would otherwise have been the multiplication g du, g om: the shift costs no instruction.
// Chunks past the end of a row that does not fill the tile are skipped.
// WIDTH_ONLY = the caps are known to be inactive for this row (alpha_l = alpha_u = 1), so
// delta_i = w_i and only the sums of gw are needed.
// SPLIT = see fuse_parts.
// MASK = the row does not fill the tile: slots past its end contribute nothing (they hold e = 0, which would
// otherwise enter as 0 - k).  base, step: see slot_base.  FULL = the first vectors of every lane, which all rows fill.
//
// Small probabilities (WIDTH_ONLY instances).  The raw width per unit of e,
//   G(x) = (1 - x) / ((1 + (a-1) x)(1 - (1-b) x)),   gw = e G(x),
// is a smooth function of x alone, and almost every token of a large vocabulary has a tiny x.  Where all the
// tokens that one instruction of the wave covers (64 lanes x one 16-byte vector) stay below the bound x_thr the
// host has fitted for this call's radius, G comes from a degree-4 polynomial 1 + x P(x) (relative error <= 2e-8,
// below the rounding of the rational form) instead of three FMAs, a product and a reciprocal: five instruction
// issues instead of ten.  The test costs half an issue per token (a running maximum and one compare per vector).
struct WidthPoly { float d0, d1, d2, d3, ethr; };   // gw = e (1 + e (d0 + e (d1 + e (d2 + e d3)))) for e <= ethr

template <int THREADS, int NVEC, int EPV, bool WIDTH_ONLY, bool SPLIT, bool MASK, int FULL = 0>
__device__ __forceinline__ void fuse_sums(const float (&e)[NVEC * EPV], const FuseRow& fr_in, const WidthPoly& wp,
                                          const Shift& sh, int V, int base, int step, double (&q5)[5])
{
    auto live_slot = [&](int j, int k) { return j * THREADS * EPV + base + (k & ~3) + step * (k & 3) < V; };
    // The caller branches between several instances of this pass.  The row constants go through an empty asm
    // so that each instance has its own: otherwise the optimiser hoists the sub-expressions the instances share
    // (1 + cu e for every token of the lane) above the branch and spills them.
    FuseRow fr = fr_in;
    asm volatile("" : "+v"(fr.cu), "+v"(fr.nih));
    // The sums run in fp64 from the first add (fp64 adds and FMAs issue at the fp32 rate on this chip): one
    // token can hold almost all of a sum.
    double a0[2] = {0.0, 0.0}, a1[2] = {0.0, 0.0}, a2[2] = {0.0, 0.0}, a3[2] = {0.0, 0.0}, a4[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NVEC; ++j) {
        if (j >= FULL && j * THREADS * EPV >= V) continue;         // uniform: the chunk holds no token
        if constexpr (WIDTH_ONLY) {
            // e >= 0: the order of the floats is the order of their bit patterns (integer maxima need no
            // canonicalisation of their operands); a negative bound compares below every e
            int big = __float_as_int(e[j * EPV]);
#pragma unroll
            for (int k = 1; k < EPV; ++k) big = max(big, __float_as_int(e[j * EPV + k]));
            if (__builtin_amdgcn_ballot_w64(big > __float_as_int(wp.ethr)) == 0) {   // uniform over the wave
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    const float ek = e[j * EPV + k];
                    const float G = fmaf(fmaf(fmaf(fmaf(wp.d3, ek, wp.d2), ek, wp.d1), ek, wp.d0), ek, 1.0f);
                    float sw = fmaf(ek, G, -sh.kw);
                    if (MASK && j >= FULL && !live_slot(j, k)) sw = 0.f;
                    const double dw = (double)sw;
                    a1[k & 1] += dw;
                    a3[k & 1] = fma(dw, dw, a3[k & 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
                continue;
            }
        }
#pragma unroll
        for (int k = 0; k < EPV; ++k) {
            float g, du, om;
            fuse_parts<SPLIT>(e[j * EPV + k], fr, g, du, om);
            const bool live = !MASK || j < FULL || live_slot(j, k);
            float sw = fmaf(g, om, -sh.kw);
            if (!live) sw = 0.f;
            const double dw = (double)sw;
            a1[k & 1] += dw;
            a3[k & 1] = fma(dw, dw, a3[k & 1]);
            if constexpr (!WIDTH_ONLY) {
                float sl = fmaf(g, du, -sh.kl);
                if (!live) sl = 0.f;
                const double dl = (double)sl;
                a0[k & 1] += dl;
                a2[k & 1] = fma(dl, dl, a2[k & 1]);
                a4[k & 1] = fma(dl, dw, a4[k & 1]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);                         // one vector at a time: bounded working set
    }
    q5[0] = a0[0] + a0[1];
    q5[1] = a1[0] + a1[1];
    q5[2] = a2[0] + a2[1];
    q5[3] = a3[0] + a3[1];
    q5[4] = a4[0] + a4[1];
}

// Pass C for calls with a wide radius (see wide_radius): the five shifted sums and the complements
// ec_i = 1 - width_i over the tokens that exist: q[5] = sum (ec - kc), q[6] = sum (ec - kc)^2, q[7] = the
// lane's largest ec.
template <int THREADS, int NVEC, int EPV>
__device__ __forceinline__ void fuse_sums_wide(const float (&e)[NVEC * EPV], const FuseRow& fr, const Shift& sh,
                                               int V, int base, int step, double (&q)[8])
{
    double acc[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    float big = 0.f;
#pragma unroll
    for (int j = 0; j < NVEC; ++j) {
        if (j * THREADS * EPV >= V) continue;                      // uniform: the chunk holds no token
#pragma unroll
        for (int k = 0; k < EPV; ++k) {
            float gl, gw, ec;
            fuse_token_wide(e[j * EPV + k], fr, gl, gw, ec);
            if (j * THREADS * EPV + base + (k & ~3) + step * (k & 3) < V) {
                const double dl = (double)(gl - sh.kl), dw = (double)(gw - sh.kw), dc = (double)(ec - sh.kc);
                acc[0] += dl; acc[1] += dw;
                acc[2] = fma(dl, dl, acc[2]); acc[3] = fma(dw, dw, acc[3]); acc[4] = fma(dl, dw, acc[4]);
                acc[5] += dc; acc[6] = fma(dc, dc, acc[6]);
                big = fmaxf(big, ec);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) q[i] = acc[i];
    q[7] = (double)big;
}

// Pass C for a handful of tokens (V <= kTinyVocab), in fp64 from the fp32 e_i.  With so few tokens the widths
// are O(1) and Sigma can be an exact zero (two tokens: delta_1 = delta_2 identically, because x_1 + x_2 = 1
// holds for the computed x as well); fp32 token arithmetic leaves ~1e-7 there, fp64 keeps the symmetry.
// Same units as fuse_sums / fuse_sums_rad: gl, gw per token with p^l = Bc gl, p^u - p^l = Wc gw; the shift
// (the values of the row's first token, which lane 0 of wave 0 holds) is returned in kq.
// WIDE: also the complement sums of fuse_sums_wide; first_tok = index of the lane's first token.
template <typename T, int EPV, bool RAD, bool WIDE>
__device__ __forceinline__ void fuse_sums_tiny(const float (&e)[EPV], const u32x4& rad, double S_units, double a,
                                               double b, double kappa, double rmax, int first_tok, int V,
                                               double (&q5)[WIDE ? 8 : 5], double (&kq)[3])
{
    float raw[EPV];
    Elt<T>::unpack(rad, raw);
    const double invS = 1.0 / S_units;
    auto token = [&](float ef, float rawf, double& gl, double& gw, double& ec) {
        const double ed = (double)ef, x = ed * invS;
        double ak = a, bk = b;
        if constexpr (RAD) {
            const double r = radius_of((double)rawf, kappa, rmax);
            ak = exp(r); bk = exp(-r);
        }
        const double om = 1.0 - x, du = 1.0 + (ak - 1.0) * x, dl = bk + (1.0 - bk) * om;   // dl = 1 - (1-b) x
        gl = ed / dl; gw = ed * om / (du * dl);
        if constexpr (RAD) { gl *= bk; gw *= ak - bk; }
        ec = (1.0 - 2.0 * (1.0 - bk) * x * om) / (du * dl);
    };
    // the same reference in every lane: lane 0's first token
    const float e_ref = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(e[0])));
    const float raw_ref = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(raw[0])));
    token(e_ref, raw_ref, kq[0], kq[1], kq[2]);
#pragma unroll
    for (int i = 0; i < (WIDE ? 8 : 5); ++i) q5[i] = 0.0;
#pragma unroll
    for (int k = 0; k < EPV; ++k) {
        if (first_tok + k < V) {
            double gl, gw, ec;
            token(e[k], raw[k], gl, gw, ec);
            gl -= kq[0]; gw -= kq[1];
            q5[0] += gl; q5[1] += gw;
            q5[2] = fma(gl, gl, q5[2]); q5[3] = fma(gw, gw, q5[3]); q5[4] = fma(gl, gw, q5[4]);
            if constexpr (WIDE) {
                q5[7] = fmax(q5[7], ec);
                ec -= kq[2];
                q5[5] += ec; q5[6] = fma(ec, ec, q5[6]);
            }
        }
    }
}

// Pass C in tensor-radius mode: every token has its own a_i, b_i from the raw radius row `rad` (as loaded,
// padding already zeroed); the sums are of p^l_i S and (p^u_i - p^l_i) S themselves, about the shift sh.
// WIDE: also the complement sums of fuse_sums_wide.
// UNIT = the radius scale is 1 (see radius_am1).
// The raw radius of a row's token above 1/2, picked up on the way: looked for in the wave that holds the row's largest
// token, by that token's e.  (No other token has it: two of them would be all of S.)
struct TopToken { bool search, found; float e, raw; };             // search: uniform over the wave; found: this lane's
template <typename T, int THREADS, int NVEC, bool WIDE, bool UNIT>
__device__ __forceinline__ void fuse_sums_rad(const float (&e)[NVEC * Elt<T>::kPerVec], const u32x4 (&rad)[NVEC],
                                              const FuseRow& fr, const RadiusMode& rm, const Shift& sh, int V,
                                              int tid, double (&q5)[WIDE ? 8 : 5], TopToken& top)
{
    const float kappa = rm.kappa, rmax = rm.rmax, am1_max = rm.am1_max;
    constexpr int EPV = Elt<T>::kPerVec;
    double a0[2] = {0.0, 0.0}, a1[2] = {0.0, 0.0}, a2[2] = {0.0, 0.0}, a3[2] = {0.0, 0.0}, a4[2] = {0.0, 0.0};
    double c1 = 0.0, c2 = 0.0;
    float big = 0.f;
#pragma unroll
    for (int j = 0; j < NVEC; ++j) {
        if (j * THREADS * EPV >= V) continue;                      // uniform: the chunk holds no token
        float raw[EPV];
        Elt<T>::unpack(rad[j], raw);
#pragma unroll
        for (int k = 0; k < EPV; ++k) {
            float pl, w;
            const bool live = (j * THREADS + tid) * EPV + k < V;
            if constexpr (WIDE) {
                float ec;
                fuse_token_rad_wide<T, UNIT>(e[j * EPV + k], raw[k], fr, kappa, rmax, am1_max, pl, w, ec);
                if (live) {
                    const double dc = (double)(ec - sh.kc);
                    c1 += dc; c2 = fma(dc, dc, c2);
                    big = fmaxf(big, ec);
                }
            } else {
                fuse_token_rad<T, UNIT>(e[j * EPV + k], raw[k], fr, kappa, rmax, am1_max, pl, w);
            }
            const double dl = live ? (double)(pl - sh.kl) : 0.0, dw = live ? (double)(w - sh.kw) : 0.0;
            a0[k & 1] += dl;
            a1[k & 1] += dw;
            a2[k & 1] = fma(dl, dl, a2[k & 1]);
            a3[k & 1] = fma(dw, dw, a3[k & 1]);
            a4[k & 1] = fma(dl, dw, a4[k & 1]);
        }
        if (top.search) {
#pragma unroll
            for (int k = 0; k < EPV; ++k) {
                const bool is = e[j * EPV + k] == top.e;
                top.raw = is ? raw[k] : top.raw;
                top.found = top.found || is;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    q5[0] = a0[0] + a0[1];
    q5[1] = a1[0] + a1[1];
    q5[2] = a2[0] + a2[1];
    q5[3] = a3[0] + a3[1];
    q5[4] = a4[0] + a4[1];
    if constexpr (WIDE) { q5[5] = c1; q5[6] = c2; q5[7] = (double)big; }
}

// Whether a second row fits in the registers at four waves per SIMD next to the centre row's floats (fp32 tiles of
// up to 8 vectors per lane) ...
// ... during the interval pass, so that the verifier row can be requested ahead of it (scalar radius: with a radius
// tensor that place is taken by the raw radius row);
template <typename T, int THREADS, int NVEC, bool DO_V, bool RAD, bool WIDE>
constexpr bool second_row_early()
{
    return DO_V && !RAD && !WIDE && !next_by_lds<T, THREADS, NVEC, DO_V, RAD, WIDE>() && (NVEC * Elt<T>::kPerVec + NVEC * 4 + 56) * 4 <= 512;
}
// ... behind it, so that a launch with a verifier row makes the residual draws of its rejected rows inside the
// streaming kernel (scalar or tensor radius: by then the verifier row has taken the raw radius row's place).
template <typename T, int THREADS, int NVEC, bool DO_V, bool RAD, bool WIDE>
constexpr bool draws_in_stream()
{
    return (DO_V && next_by_lds<T, THREADS, NVEC, DO_V, RAD, WIDE>()) || (DO_V && !WIDE && (NVEC * Elt<T>::kPerVec + NVEC * 4 + 56) * 4 <= 512);
}
// Most rows a workgroup has room for: kMaxRowsPerWg, or what the rows in flight leave of a compute unit's LDS.
template <typename T, int THREADS, int NVEC, bool DO_V, bool RAD, bool WIDE>
constexpr int rows_per_wg()
{
    return !next_by_lds<T, THREADS, NVEC, DO_V, RAD, WIDE>() || THREADS >= 512 ? kMaxRowsPerWg : THREADS == 256 ? 64 : THREADS == 128 && NVEC > 8 ? 40 : 16;
}
// Workgroups of an instance on a compute unit.  The register budget the kernel was compiled for fixes how many fit: target_waves()
// waves per SIMD, and a workgroup puts THREADS / 256 waves on each of the four SIMDs (a 128-lane one: one wave on two of them).
// Where rows come through LDS, no more than its LDS has room for, and as many waves on every SIMD: 12 of 64 lanes and eight vectors.
// (Quantified, on a grid for the 16 that the registers allow / for 14, which fit / for 12: 16384 x 4096 bf16 49.9 / 43.9 / 40.1 us,
// 9000 x 4096 32.2 / 28.6 / 26.8, 60000 x 4096 150 / 141 / 142; fp32 4096 x 2048 - / 14.5 / 13.2.)  The arrays in LDS are counted as the
// kernel declares them; tests/test_resources.py holds the result against the built kernels.
template <typename T, int THREADS, int NVEC, bool DO_Q, bool DO_V, bool RAD, bool WIDE>
constexpr int workgroups_per_unit()
{
    constexpr int by_waves = target_waves<T, THREADS, NVEC, RAD, DO_V>() * 256 / THREADS;
    if (!next_by_lds<T, THREADS, NVEC, DO_V, RAD, WIDE>()) return by_waves;
    constexpr int NW = THREADS / 64, rows = rows_per_wg<T, THREADS, NVEC, DO_V, RAD, WIDE>();
    constexpr int in_flight = THREADS * NVEC * 16;                                                   // sm_next
    constexpr int waves = NW * (16 + 16 + 512 + (DO_Q ? 80 : 0) + (DO_V ? 8 + 16 : 0)) + 24;         // sm_ref2 ... sm_sum, sm_k
    constexpr int parked = rows * ((int)sizeof(RowStats) + 16 + (DO_V ? 4 + 4 + 1 : 0));             // sm_rows ... sm_close
    constexpr int draws = DO_V ? NW * (NVEC * 8 + 1024 + 4 + 4) : 0;                                 // sm_tab, sm_quad, sm_auxf, sm_auxi
    constexpr int even = THREADS < 256 ? 256 / THREADS : 1;
    constexpr int by_lds = lds_fit(in_flight + waves + parked + draws) / even * even;
    return by_lds < by_waves ? by_lds : by_waves;
}

// sm_draw / row_id of a rejected row whose draw is still to be made (by resample_kernel)
constexpr int kDrawPending = -2;

// A condition with what it is expected to be, in the instances where `hint` is true.  (A macro: said inside a function, the expectation
// is lost before the function is inlined.)
#define CIAR_USUAL(hint, c) ((hint) ? __builtin_expect(!!(c), 1) : !!(c))
#define CIAR_RARE(hint, c) ((hint) ? __builtin_expect(!!(c), 0) : !!(c))

// WHOLE: every row fills the tile.  Such calls have instances of their own, without the code for rows that do not (vectors past the
// end clamped, tokens masked): a call of a few rows waits for its instructions to arrive, and longer for those behind a jump (8 x
// 16384 fp32 13.8 -> 13.0 us, 256 rows 16.1 -> 15.5, 2048 rows 51.5 -> 50.4).  The others tell at run time: with masks that are
// wanted in any case the compiler forms them ahead of the row loop and spills them (up to 500 B).
template <typename T, int THREADS, int NVEC, bool DO_Q, bool DO_V, bool RAD, bool WIDE, bool WHOLE>
__global__ __launch_bounds__(THREADS)
__attribute__((amdgpu_waves_per_eu(target_waves<T, THREADS, NVEC, RAD, DO_V>())))
void stream_kernel(const RowArgs A)
{
    using E = Elt<T>;
    constexpr int EPV = E::kPerVec;
    constexpr int EPT = NVEC * EPV;
    constexpr int NW = THREADS / 64;
    constexpr int CHUNK = THREADS * EPV;            // tokens covered by one load instruction of the workgroup
    constexpr bool LDS_NEXT = next_by_lds<T, THREADS, NVEC, DO_V, RAD, WIDE>();
    // The verifier row is requested before the interval pass where a second row fits in the registers at
    // four waves per SIMD next to the centre row's floats (fp32 tiles of up to 8 vectors per lane; measured
    // 51 -> 48.6 us on the benchmark); elsewhere it would spill, and it is requested after the pass.
    constexpr bool EARLY_T = second_row_early<T, THREADS, NVEC, DO_V, RAD, WIDE>();
    // Quantify-only launches have no verifier row; under the same condition the next centre row is requested
    // before the interval pass instead.
    constexpr bool EARLY_NEXT = !DO_V && !RAD && !WIDE && !LDS_NEXT && (EPT + NVEC * 4 + 56) * 4 <= 512;
    // A rejected row's draw needs both rows.  Where two rows fit, the centre row's exponentials simply stay in their
    // registers next to the verifier row and the draw is made here (KEEP_E).  Elsewhere (bf16 tiles of eight vectors, the 16-vector
    // fp32 tile, wide radii) the two do not fit: such rows are only marked, and resample_kernel
    // draws them behind this kernel (measured with the draw here and the centre row fetched again: the branch
    // alone, never taken, cost the bf16 row loop 11 % -- registers and scheduling -- and workload 3 ran 318 against
    // 285 us per step).
    constexpr bool KEEP_E = draws_in_stream<T, THREADS, NVEC, DO_V, RAD, WIDE>();
    constexpr int ROWS = rows_per_wg<T, THREADS, NVEC, DO_V, RAD, WIDE>();
    constexpr int FULL = full_vectors<T, THREADS, NVEC, DO_V, RAD, WIDE>();
    // bf16 rows go through the matrix cores (see bf16_scaled; with a radius tensor the verifier row only) where a lane holds enough of
    // a row for it to pay: with one or two vectors a row is a chain of latencies (871 x 1162 verified 10.2 us without, 10.7 with).
    constexpr bool MATRIX_T = sizeof(T) == 2 && NVEC >= 4, MATRIX = MATRIX_T && !RAD;
    constexpr int NQ = WIDE ? 8 : 5;                // interval sums a wave hands over
    // A row with a token above 1/2 and a radius tensor: finish_row wants that token's raw radius.  It is picked up in the
    // interval pass -- except in the instances of 1024 lanes with bf16 rows, which spill: there only the token's index is
    // parked, ahead of the pass, and the finishing lane fetches its radius (picked up in the pass: 1017 rows of 65536 tokens
    // 157 us against 148, 1666 of 40000 288 against 268; the other instances lose up to 9 % by the index).
    constexpr bool TOP_INDEX = RAD && sizeof(T) == 2 && THREADS == 1024;
    constexpr int NT = NVEC * NW;                   // pieces of a row in token order: (vector j, wave w) -> j NW + w

    // Exchange slots.  Two barriers per row order every write against every read: the centre-row
    // slots are written before the first and read between the two, the others are written between the
    // two and read after the second, before the next row's first barrier.
    // (the centre-row slots exist twice and rows alternate between them: a row's write-up and its draw read them
    // after the second barrier, when a wave that runs ahead may already be writing the next row's)
    __shared__ float  sm_ref2[2][NW * 2];           // per wave: max centre logit, n_w
    __shared__ double sm_S2[2][NW];                 // per wave: S_w
    // (LDS_NEXT, where a row has one barrier: these exist twice as well)
    __shared__ float  sm_nt2[LDS_NEXT ? 2 : 1][NW]; // per wave: nt_w
    __shared__ double sm_Z2[LDS_NEXT ? 2 : 1][NW];  // per wave: Z_w
    __shared__ double sm_q52[LDS_NEXT ? 2 : 1][NW * NQ];   // per wave: the interval sums, already in row units
    __shared__ double sm_sum[LDS_NEXT ? NW : 1][LDS_NEXT ? 64 : 1];       // LDS_NEXT, per wave: [interval sums of the row before, S_w, Z_w][eight groups of lanes]
    __shared__ double sm_k[3];                      // the shift the sums are taken about (row units), from wave 0
    __shared__ float  sm_e0;                        // e of the row's first token, in the units of wave 0
    // Finishing inside this kernel: the statistics of the rows this workgroup has streamed since its last
    // finishing step (at most ROWS of them) and, fetched ahead, what their finishing needs from memory:
    // the reported token's centre logit, raw radius and verifier logit, the row's two uniforms.
    __shared__ RowStats sm_rows[ROWS];
    __shared__ float    sm_fx[ROWS][4];    // cx, rawx, tx, u_accept
    __shared__ float    sm_rtop[RAD && !TOP_INDEX ? ROWS : 1];   // raw radius of the row's token above 1/2, if any
    __shared__ int      sm_top[TOP_INDEX ? ROWS : 1];            // or its index
    __shared__ float    sm_ur[DO_V ? ROWS : 1];
    __shared__ int      sm_draw[DO_V ? ROWS : 1];   // -1: the drafted token was accepted; else the row's draw
    __shared__ uint8_t  sm_close[DO_V ? ROWS : 1];  // the fp32 accept test could not decide the row
    __shared__ double   sm_tab[DO_V ? NT : 1];      // residual mass of each piece of a rejected row
    __shared__ __attribute__((aligned(16))) double sm_quad[KEEP_E && (NVEC >= 8 || LDS_NEXT) ? NW : 1][KEEP_E && (NVEC >= 8 || LDS_NEXT) ? 8 : 1][16];   // a draw's quad sums
    __shared__ float    sm_auxf[DO_V ? NW : 1];
    extern __shared__ u32x4 sm_next[];              // LDS_NEXT: [NVEC][THREADS], the row in flight, centre and verifier row in turn
    __shared__ int      sm_auxi[DO_V ? NW : 1];

    const int tid = threadIdx.x, lane = tid & 63;
    // (uniform over the wave; bf16 instances keep it in a scalar register, so that nothing indexed by it -- the waves'
    // exchange slots in LDS -- is held in vector registers across the row loop: they have none to spare.  The fp32
    // instances measured 1 % slower that way.)
    const int wave = THREADS == 64 ? 0 : sizeof(T) == 2 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
    const int V = A.V;
    RadiusMode rm = {false, 0.f, 0.f, 0.f};
    if constexpr (RAD) {
        rm = radius_mode(A);
        // (in scalar registers; the fp32 instances of eight and sixteen waves spill with it)
        if constexpr (sizeof(T) == 2 || THREADS == 256) { rm.kappa = uniform_f(rm.kappa); rm.rmax = uniform_f(rm.rmax); rm.am1_max = uniform_f(rm.am1_max); }
    }
    // What the branches expect decides what lies next to each other, and what the register allocator favours.  Not expected:
    // anything, where ragged rows are one vector to a lane (or two, bf16): 2048 x 1023 fp32 fused 16.6 us with, 16.3 without, 2048 x
    // 2500 bf16 23.3 and 22.4; the inactive caps in fp32 calls with a verifier row: eight vectors to a lane spill 12 to 76 B with it (2048
    // x 5000 28.7 and 28.5; quantify-only 2048 x 2500 wants it, 12.0 and 12.7); the draws' usual course in fp32 on ragged rows of 1024 lanes
    // (36 B; 2048 x 20001 95.6 and 94.7).
    constexpr bool FP32_V = sizeof(T) == 4 && DO_V && !RAD;
    constexpr bool HINTS = RAD || WHOLE || (sizeof(T) == 2 ? NVEC >= 4 : NVEC > 1 || !DO_V);
    constexpr bool HINT_CAPS = HINTS && !FP32_V, HINT_DRAW = HINTS && !(FP32_V && THREADS == 1024 && !WHOLE);
    // bf16: what is formed from the thread's index -- masks, slots' addresses -- is formed anew for every row, from an opaque copy of
    // it, where it would otherwise be held, or spilled, through the row loop.  (Not in calls with one row of few vectors: there is
    // room to hold it, 2048 x 1162 verified 14.9 us so, 15.1 otherwise.)
    constexpr bool FORM_ANEW = sizeof(T) == 2 && (MATRIX_T || RAD || (DO_Q && DO_V));
    const bool partial = !WHOLE && V != NVEC * CHUNK;              // uniform: the row does not fill the tile
    const int last_vec = (V + EPV - 1) / EPV - 1;
    const int nrows = (int)A.N;
    const int step = (int)gridDim.x;

    // Rows live in global memory (address space 1).  Vector j of this lane: scalar row base + 32-bit
    // byte offset.  A row that fills the tile needs one lane offset for all of its vectors (the
    // distance between vectors is a constant on top of the scalar base).  Otherwise vector indices
    // past the end of the row are clamped to its last vector, so every lane loads valid memory
    // unconditionally; tokens that do not exist are set to -inf afterwards.
    // The loads are non-temporal: every logit is used exactly once, and streaming past the caches measured
    // 10-12 % more bandwidth than ordinary loads on this chip (plain read of 2 GiB: 6.2 -> 6.9 TB/s).
    // The base goes through readfirstlane and the lane index through an empty asm: both are opaque
    // to the optimiser, which otherwise turns the sixteen addresses of a row into sixteen 64-bit
    // induction variables, spills them, and serialises the loads on the reloads.
    // `whole` = false: every lane fetches the row's first vectors only (a few cache lines per wave, results unused).
    // The quantify-only loop requests its next row this way when there is none: a request under a branch made the
    // register allocator spill a third of the centre row there (none when the request is unconditional).
    auto load_row = [&](u32x4 (&buf)[NVEC], const void* rows, int r, bool whole = true) {
        const uint64_t b = (uint64_t)(static_cast<const T*>(rows) + row_offset(A, r));
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
        const gbytes base = (gbytes)(((uint64_t)hi << 32) | lo);
        int t = whole ? tid : 0;
        asm volatile("" : "+v"(t));
        if (partial) {
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
                const uint32_t off = (uint32_t)min(j * THREADS + t, last_vec) * 16u;
                buf[j] = __builtin_nontemporal_load((gvec)(base + off));
            }
        } else {
            const uint32_t off = (uint32_t)t * 16u;
#pragma unroll
            for (int j = 0; j < NVEC; ++j) buf[j] = __builtin_nontemporal_load((gvec)(base + (uint64_t)j * (THREADS * 16u) + off));
        }
    };
    // A row into LDS (lane l of a wave lands 16 l bytes behind the address the wave names; a lane reads back only what
    // its own wave has requested).
    auto fetch_row = [&](const void* rows, int r) {
        using lds_ptr = __attribute__((address_space(3))) void*;
        using glb_ptr = const __attribute__((address_space(1))) void*;
        const uint64_t b = (uint64_t)(static_cast<const T*>(rows) + row_offset(A, r));
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
        const gbytes base = (gbytes)(((uint64_t)hi << 32) | lo);
        const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
        int t = tid;
        asm volatile("" : "+v"(t));
        const uint32_t off = (uint32_t)t * 16u;
#pragma unroll
        for (int j = 0; j < NVEC; ++j) {
            if (partial)
                __builtin_amdgcn_global_load_lds((glb_ptr)(base + (uint32_t)min(j * THREADS + t, last_vec) * 16u),
                                                 (lds_ptr)(sm_next + j * THREADS + w * 64), 16, 0, kNonTemporal);
            else
                __builtin_amdgcn_global_load_lds((glb_ptr)(base + (uint64_t)j * (THREADS * 16u) + off),
                                                 (lds_ptr)(sm_next + j * THREADS + w * 64), 16, 0, kNonTemporal);
        }
    };
    // the row in flight has landed and moves to registers
    auto take_row = [&](u32x4 (&buf)[NVEC]) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int t = tid;
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int j = 0; j < NVEC; ++j) buf[j] = sm_next[j * THREADS + t];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // The sums of a wave reduced together: every lane's value -> groups of eight lanes (three DPP steps) -> LDS; then lane l takes
    // quantity l / 8 and three more steps finish all eight (LDS operations of a wave complete in order: no barrier).
    auto sum_of_eight = [](double v) {
        v = dpp_add<0xB1, 0xf>(v);                                 // lane ^ 1  (quad_perm 1,0,3,2)
        v = dpp_add<0x4E, 0xf>(v);                                 // lane ^ 2  (quad_perm 2,3,0,1)
        return dpp_add<0x141, 0xf>(v);                             // the other quad of the eight (row_half_mirror)
    };
    auto put_sum = [&](double v, int which, int l) {
        v = sum_of_eight(v);
        if ((l & 7) == 0) sm_sum[LDS_NEXT ? wave : 0][which * 8 + (l >> 3)] = v;
    };
    auto get_sums = [&](int l) { return sum_of_eight(sm_sum[LDS_NEXT ? wave : 0][l < 56 ? l : 0]); };
    // wave 0: a row's interval sums over the waves
    auto park_sums_of = [&](int at, int p) {
        int l = tid;
        asm volatile("" : "+v"(l));
        if (l < 5) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) t += sm_q52[LDS_NEXT ? p : 0][w * NQ + l];
            const float mode = sm_rows[at].mode;
            const bool width_only = mode == kSumsWidthOnly || mode == kSumsWidthOnly + kSumsFlatPending;
            sm_rows[at].q[l] = width_only && l != 1 && l != 3 ? 0.0 : t;   // (its other slots hold what an earlier row left)
        }
    };
    // (__syncthreads would wait for that row as well)
    auto row_barrier = [&]() {
        if constexpr (LDS_NEXT) lds_barrier();
        else __syncthreads();
    };
    // (constants of the matrix cores' products are formed where they are used, from an opaque copy of the thread index: an
    // instruction or two per register and row, where they would otherwise be held through the row loop)
    auto opaque_tid = [&]() {
        int t = tid;
        asm volatile("" : "+v"(t));
        return t;
    };
    auto mask_with = [&](u32x4& r, int first, uint32_t fill) {
        if constexpr (sizeof(T) == 2) E::mask_tail(r, first, V, fill);
        else E::mask_tail(r, first, V);
    };
    // Verifier row statistics of one wave from the row as loaded: nt_w and Z_w = sum 2^(t_i log2e - nt_w).
    // Any integer reference serves as long as no term overflows and the large terms stay normal numbers, so the
    // sum is first taken about the reference of the centre row's tokens in the same wave (`guess`: verifier
    // logits follow the device model's), which saves the pass for the maximum; a sum outside [2^-40, 2^100]
    // (a verifier row far from its centre row, or a wave without tokens: sum 0) is redone about the wave's own
    // maximum.
    auto verifier_mask = [&](u32x4 (&tb)[NVEC], uint32_t fill) {
        if (partial) {
            const int ot = FORM_ANEW ? opaque_tid() : tid;
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
                if (!LDS_NEXT || (j + 1) * CHUNK > V) mask_with(tb[j], (j * THREADS + ot) * EPV, fill);
            }
        }
    };
    // (the lane's share of the sum about the reference nref; quads: the tokens widened by the matrix cores)
    auto verifier_lane_sum = [&](u32x4 (&tb)[NVEC], float nref, bool quads) {
        float zacc[4] = {0.f, 0.f, 0.f, 0.f};
        // (LDS_NEXT, where a lane holds more of a row: a vector's tokens in fp32, the vectors in fp64)
        double zsum = 0.0;
        auto add_vector = [&](float (&t)[EPV]) {
#pragma unroll
            for (int w = EPV / 2; w > 0; w /= 2) {
#pragma unroll
                for (int k = 0; k < w; ++k) t[k] += t[k + w];
            }
            zsum += (double)t[0];
        };
        if constexpr (MATRIX_T) {
            if (quads) {
                const Bf16Scale bs = bf16_scale(opaque_tid());
                float z[2][EPV];
                bf16_scaled(tb[0], bs, z[0]);
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    if (j + 1 < NVEC) bf16_scaled(tb[j + 1], bs, z[(j + 1) & 1]);   // (the matrix cores one vector ahead)
                    if constexpr (LDS_NEXT) {
                        float t[EPV];
#pragma unroll
                        for (int k = 0; k < EPV; ++k) t[k] = exp2_scaled(z[j & 1][k], nref);
                        add_vector(t);
                    } else {
#pragma unroll
                        for (int k = 0; k < EPV; ++k) zacc[k & 3] += exp2_scaled(z[j & 1][k], nref);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (LDS_NEXT) return zsum;
                else return (double)((zacc[0] + zacc[1]) + (zacc[2] + zacc[3]));
            }
        }
#pragma unroll
        for (int j = 0; j < NVEC; ++j) {
            float tv[EPV];
            E::unpack(tb[j], tv);
            if constexpr (LDS_NEXT) {
#pragma unroll
                for (int k = 0; k < EPV; ++k) tv[k] = E::exp2_ref(tv[k], nref);
                add_vector(tv);
            } else {
#pragma unroll
                for (int k = 0; k < EPV; ++k) zacc[k & 3] += E::exp2_ref(tv[k], nref);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (LDS_NEXT) return zsum;
        else return (double)((zacc[0] + zacc[1]) + (zacc[2] + zacc[3]));
    };
    // (the sum about the guess was out of range: about the wave's own maximum -- after a second look without the matrix cores
    // where a masked token can have got into the way)
    // (`quads` is false afterwards)
    auto verifier_redo = [&](u32x4 (&tb)[NVEC], float& ntw, double& Zw, bool& quads) {
        auto in_range = [&]() { return Zw >= 0x1p-40 && Zw <= 0x1p100; };   // (false for NaN)
        if constexpr (sizeof(T) == 2) {
            if (CIAR_RARE(HINTS, quads && !in_range())) {                            // uniform over the wave
                quads = false;
                verifier_mask(tb, E::kNegInfWord);
                Zw = wave_sum(verifier_lane_sum(tb, ntw, false));
            }
        }
        if (CIAR_RARE(HINTS, !in_range())) {                // uniform over the wave
            float mt = -INFINITY;
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
                float tv[EPV];
                E::unpack(tb[j], tv);
#pragma unroll
                for (int k = 0; k < EPV; ++k) mt = fmaxf(mt, tv[k]);
            }
            ntw = ref_of(wave_max(mt));
            Zw = wave_sum(verifier_lane_sum(tb, ntw == -INFINITY ? 0.f : ntw, false));   // an all-masked wave: every term is 2^-inf = 0
        }
    };
    auto verifier_stats = [&](u32x4 (&tb)[NVEC], float guess, float& ntw, double& Zw, bool& quads) {
        verifier_mask(tb, quads ? kNoTokenWord : E::kNegInfWord);
        ntw = guess == -INFINITY ? 0.f : guess;
        Zw = wave_sum(verifier_lane_sum(tb, ntw, quads));
        verifier_redo(tb, ntw, Zw, quads);
    };

    // ---- which rows this workgroup takes ---------------------------------------------------------------------
    // Pieces of `unit` consecutive rows: piece blockIdx.x, blockIdx.x + gridDim.x, ...  (unit = 1, or the window
    // length when this kernel also writes the window outputs).  The workgroup's rows are numbered L = 0, 1, 2, ...
    // in the order it streams them; with finishing there are at most `cap` of them (whole pieces; the launcher sizes
    // the grid accordingly), and after the last one one lane per row finishes it from what is parked in LDS.
    const bool finish = (DO_V || A.finish) && (DO_Q || DO_V);      // uniform over the grid
    const int unit = DO_V ? A.unit : 1;
    const int cap = (ROWS / unit) * unit;
    auto row_of = [&](int L) -> int64_t {
        const int u = L / unit;
        return ((int64_t)blockIdx.x + (int64_t)u * step) * unit + (L - u * unit);
    };
    // What the finishing of rows L0 ... L0 + cap - 1 needs from memory (lane t: row L0 + t), in three steps so that
    // the first row's own loads can go in between: fetch_ids requests the reported tokens, fetch_scalars (which
    // waits for them) their logits and the uniforms, park_scalars (which waits for those) leaves them in LDS.
    struct RowScalars { float cx, rawx, tx, ua, ur; bool live; };
    auto fetch_ids = [&](int L0) {
        const int64_t r = row_of(L0 + tid);
        return (tid < cap && r < nrows && A.ids) ? A.ids[ids_index(A, r)] : 0;
    };
    auto fetch_scalars = [&](int L0, int xid) {
        RowScalars f = {0.f, 0.f, 0.f, 0.f, 0.f, false};
        const int64_t r = row_of(L0 + tid);
        if (tid < cap && r < nrows) {
            f.live = true;
            if (A.ids) {
                xid = xid < 0 ? 0 : (xid >= V ? V - 1 : xid);
                f.cx = load_logit(static_cast<const T*>(A.draft) + row_offset(A, r), xid);
                if constexpr (RAD) f.rawx = load_logit(static_cast<const T*>(A.radius) + row_offset(A, r), xid);
                if constexpr (DO_V) f.tx = load_logit(static_cast<const T*>(A.target) + row_offset(A, r), xid);
            }
            if constexpr (DO_V) { f.ua = A.u_accept[r]; f.ur = A.u_resample[r]; }
        }
        return f;
    };
    auto park_scalars = [&](const RowScalars& f) {
        if (f.live) {
            sm_fx[tid][0] = f.cx; sm_fx[tid][1] = f.rawx; sm_fx[tid][2] = f.tx; sm_fx[tid][3] = f.ua;
            if constexpr (DO_V) sm_ur[tid] = f.ur;
        }
    };
    // Finishing of the rows L0 ... L0 + cnt - 1 from what is parked in LDS, two lanes per row, from 128 lanes on in different
    // waves so that the two halves run side by side: lane i < HALF writes row i's statistics and its quantifier outputs (Eq.
    // uncertainty_score, the threshold of Algorithm 1), lane HALF + i its verification outputs; with unit == window
    // also the outputs of the windows (Algorithm 1: the verified prefix of a drafted window and the token that
    // replaces its first rejection).
    auto finish_batch = [&](int L0, int cnt) {
        constexpr int HALF = THREADS >= 256 ? 128 : THREADS / 2;
        static_assert(ROWS <= HALF, "two lanes per parked row");
        __syncthreads();
        // (the lane index through an empty asm: otherwise the row indices below are the ones fetch_scalars formed
        // before the first row, kept in registers or spilled for the whole of the row loop)
        int ft = tid;
        asm volatile("" : "+v"(ft));
        // (likewise the piece length: the divisions by it below otherwise start from what the prologue formed)
        int unit_f = unit;
        asm volatile("" : "+s"(unit_f));
        const int i = ft & (HALF - 1);                             // the parked row this lane works on
        const bool mine = ft < 2 * HALF && i < cnt;
        const bool qjob = mine && ft < HALF, vjob = DO_V && mine && ft >= HALF;
        const int64_t r = row_of(L0 + i);
        auto quantify_half = [&]() {
            if (qjob) {
                const RowStats st = sm_rows[i];
                A.stats[r] = st;
                if constexpr (DO_Q) {
                    const float cx = A.ids ? sm_fx[i][0] : st.mc;  // no ids: the arg-max token is reported
                    float raw_top = RAD && !TOP_INDEX ? sm_rtop[RAD && !TOP_INDEX ? i : 0] : 0.f;
                    if (TOP_INDEX && (double)E::exp2_ref(st.mc, st.n == -INFINITY ? 0.f : st.n) > 0.5 * st.S)
                        raw_top = load_logit(static_cast<const T*>(A.radius) + row_offset(A, r), sm_top[TOP_INDEX ? i : 0]);
                    finish_row<T, RAD>(A, r, st, cx, 0.f, sm_fx[i][1], 0.f, true, false, raw_top);
                }
            }
        };
        // (where the row loop has made the accept test and windows span workgroups, the other half has next to nothing
        // to do ahead of the barrier below and a trip to memory and back behind it -- the window arrivals: there the
        // quantify half runs behind the barrier, next to those, instead of ahead of it, where the other lanes would
        // wait for it; measured on the benchmark: 59.0 -> 57.5 us per step together with the early claim)
        const bool q_late = KEEP_E && A.win_count != nullptr;      // uniform
        if (!q_late) quantify_half();
        if constexpr (DO_V) {
            if (vjob) {
                const RowStats& st = sm_rows[i];
                if constexpr (KEEP_E) {
                    // the row loop has decided in fp32 and drawn; rows it found too close to call are decided here
                    if (sm_close[i] && !reject_exact<T>(sm_fx[i][0], sm_fx[i][2], sm_fx[i][3], st.n, st.nt, st.S, st.Z))
                        sm_draw[i] = -1;                           // accepted after all: the draw does not count
                } else {
                    // the accept test (Algorithm 1, "Cloud verification"); a rejected row's draw is resample_kernel's
                    sm_draw[i] = reject_exact<T>(sm_fx[i][0], sm_fx[i][2], sm_fx[i][3], st.n, st.nt, st.S, st.Z)
                                     ? kDrawPending : -1;
                }
            }
            __syncthreads();                                       // the windows below read their rows' final draws
            if (q_late) quantify_half();
            if (vjob) {
                const int id = sm_draw[i];                         // -1, a draw, or kDrawPending
                if (A.accept) A.accept[r] = (uint8_t)(id == -1);
                if (A.row_id) A.row_id[r] = id;
                // (an opaque copy: the reciprocal that the divisions by K below start from is otherwise the one the
                // workgroup formed for its claim ahead of the first row, kept -- spilled -- through the whole row loop)
                int K = A.window;
                asm volatile("" : "+s"(K));
                if (unit_f == K && !A.win_count && (A.accept_len || A.resampled_id) && i % K == 0) {   // pieces start at multiples of K
                    const int64_t left = nrows - r;
                    const int len = (int)(left < K ? left : K);
                    int m = 0;
                    while (m < len && sm_draw[i + m] == -1) ++m;
                    const uint32_t w = (uint32_t)r / (uint32_t)K;
                    if (A.accept_len) A.accept_len[w] = m;
                    // (a pending draw: resample_kernel writes the window's entry when it has drawn that row)
                    if (A.resampled_id && (m == len || sm_draw[i + m] != kDrawPending))
                        A.resampled_id[w] = m < len ? sm_draw[i + m] : -1;
                }
                if constexpr (KEEP_E) {
                    const int64_t w = (int64_t)((uint32_t)r / (uint32_t)K), lo = w * K;
                    if (A.win_count && (i % unit_f == 0 || r == lo)) {
                        // A window that spans workgroups: the consecutive rows of it that this workgroup holds (one
                        // row where the rows are dealt out singly: measured the fastest for such launches, 58.8 us per
                        // step on workload 2 against 63.2 us with four consecutive rows per workgroup, whose two
                        // arrivals per window cost less than their memory access pattern loses) arrive together in the
                        // window's 64-bit word (window_arrive), from the lane of the first of them, and the arrival
                        // that completes the window writes its outputs.
                        const int len = (int)(nrows - lo < K ? nrows - lo : K);
                        const int piece_end = i - i % unit_f + unit_f;
                        int rows = 0, off = 0, mine_id = -1;
                        for (; i + rows < cnt && i + rows < piece_end && r + rows < lo + len; ++rows) {
                            if (mine_id < 0 && sm_draw[i + rows] >= 0) { mine_id = sm_draw[i + rows]; off = (int)(r + rows - lo); }
                        }
                        int first, draw;
                        if (window_arrive(A.win_count + 2 * lo, A.tag, rows, off, mine_id, len, first, draw)) {
                            if (A.accept_len) A.accept_len[w] = first < 0 ? len : first;
                            if (A.resampled_id) A.resampled_id[w] = first < 0 ? -1 : draw;
                        }
                    }
                }
            }
        }
        __syncthreads();
    };

    // This workgroup's rows: its pieces are whole except possibly the very last piece of the launch.
    int my_rows;
    {
        // (in 32 bits: the entry points take fewer than 2^31 rows, and a 64-bit division is ~150 scalar instructions in
        // a chain -- three of them stood between the start of the kernel and its first request for a row)
        const uint32_t b = blockIdx.x, un = (uint32_t)unit, st = (uint32_t)step;
        const uint32_t pieces = ((uint32_t)nrows + un - 1u) / un;
        const uint32_t mine = b < pieces ? (pieces - b + st - 1u) / st : 0u;
        const bool owns_last = mine > 0u && (pieces - 1u - b) % st == 0u;
        my_rows = (int)(mine * un - (owns_last ? pieces * un - (uint32_t)nrows : 0u));
    }

    // The row index is uniform over the workgroup: keep it in a scalar register.
    // A row's centre logits are loaded and worked on first, its verifier logits second: the centre row
    // carries most of the arithmetic (both of its passes), the verifier row only a short one, so
    // little work is left when the last bytes of the launch arrive.
    // The launcher sizes the grid so that a workgroup has at most `cap` rows: they are finished after the last one,
    // when nothing of a row is held in registers any more.
    constexpr int L0 = 0;
    const int cnt = min(cap, my_rows);                             // uniform
    if (cnt <= 0) return;
    int row = __builtin_amdgcn_readfirstlane((int)row_of(L0));
    int in_piece = 0;                                              // rows of the current piece already taken
    const int piece_jump = __builtin_amdgcn_readfirstlane((step - 1) * unit + 1);   // last row of a piece -> first of the next
    // windows that span workgroups: the words this workgroup's rows will arrive in are looked at first of all (see
    // window_claim), so that the answer is back before the first row is
    unsigned long long* claim_word = nullptr;
    unsigned long long claim_seen = 0;
    if constexpr (KEEP_E) {
        if (A.win_count && tid < cnt) {
            const int64_t r = row_of(L0 + tid);
            const int64_t lo = (int64_t)((uint32_t)r / (uint32_t)A.window * (uint32_t)A.window);
            if (tid % unit == 0 || r == lo) {
                claim_word = A.win_count + 2 * lo;
                claim_seen = __hip_atomic_load(claim_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    int first_id = 0;
    if (finish) first_id = fetch_ids(L0);                          // a small load, issued ahead of the first row's
    u32x4 buf[NVEC];                                               // a row as loaded: centre and verifier row in turn
    if constexpr (LDS_NEXT) fetch_row(A.draft, row);
    else load_row(buf, A.draft, row);
    // (the logits of the reported tokens are requested behind the row, once their ids are there, and parked when
    // they arrive: that waits for the row as well, which the first pass needs anyway)
    if (finish) park_scalars(fetch_scalars(L0, first_id));
    if constexpr (KEEP_E) {
        if (claim_word) window_claim(claim_word, A.tag, claim_seen);
    }

    if constexpr (THREADS < 1024) {
        if (cnt > 1) __builtin_amdgcn_s_setprio(3);                // (see "Wave priority by progress" at the end of the loop)
    }
    for (int done = 0;; ++done) {                                  // done = rows of this batch already streamed
        const bool has_next = done + 1 < cnt;                      // uniform
        // (the rows are walked without a division: within a piece the next row, at its end the next piece)
        in_piece = in_piece + 1 == unit ? 0 : in_piece + 1;
        const int next = __builtin_amdgcn_readfirstlane(has_next ? (in_piece == 0 ? row + piece_jump : row + 1) : row);
        float raw0 = 0.f;                                          // raw radius of the row's first token
        if constexpr (RAD && DO_Q) raw0 = load_logit(static_cast<const T*>(A.radius) + row_offset(A, row), 0);

        if constexpr (LDS_NEXT) {
            // the centre row has landed; its slots take the verifier row, which arrives during B
            take_row(buf);
            if constexpr (DO_V) fetch_row(A.target, row);
            else if (has_next) fetch_row(A.draft, next);
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---- B: centre row: per-wave max, e_i = 2^(c_i log2e - n_w), S_w -------------------------------
        float e[EPT];
        float mcw, nw;
        double Sw;
        // S is accumulated in fp64 from the first add: on a nearly one-hot row the bounds of the top
        // token react to a relative error in S about five times over, and on a two-token row Sigma is
        // a difference of two nearly equal widths; even one fp32 add of two comparable terms (6e-8)
        // shows there (measured against the fp64 definition).  Adding the tokens of a 16-byte vector pairwise in
        // fp32 first (fp64 only across vectors: 0.9 instructions less per token) was tried and fails parity: where a
        // cap is active Omega = alpha_u S_u - alpha_l S_l is a small difference of numbers near 1 (0.022 from
        // 1.012 - 0.99 in the failing case), which multiplies the 1e-8 that a dominant token's vector loses by 45.
        double sacc[2] = {0.0, 0.0};
        // bf16 rows: the maximum from the packed words, the tokens widened by the matrix cores (`quads`: the slots of e[] are
        // transposed, see bf16_scaled; uniform over the wave).  Not where the slots meet a radius tensor's.
        bool quads = false;
        if constexpr (MATRIX) {
            if (partial) {
                const int ot = opaque_tid();
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    if (!LDS_NEXT || (j + 1) * CHUNK > V) mask_with(buf[j], (j * THREADS + ot) * EPV, kNoTokenWord);
                }
            }
            mcw = wave_top(top_words(buf), quads);
        }
        if (MATRIX && CIAR_USUAL(HINTS, quads)) {
            nw = ref_of(mcw);
            const Bf16Scale bs = bf16_scale(opaque_tid());
            bf16_scaled(buf[0], bs, &e[0]);
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
                if (j + 1 < NVEC) bf16_scaled(buf[j + 1], bs, &e[(j + 1) * EPV]);   // (the matrix cores one vector ahead)
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    e[j * EPV + k] = exp2_scaled(e[j * EPV + k], nw);
                    sacc[k & 1] += (double)e[j * EPV + k];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            if (partial) {
                const int ot = FORM_ANEW ? opaque_tid() : tid;
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    if (!LDS_NEXT || (j + 1) * CHUNK > V) E::mask_tail(buf[j], (j * THREADS + ot) * EPV, V);
                }
            }
#pragma unroll
            for (int j = 0; j < NVEC; ++j) E::unpack(buf[j], &e[j * EPV]);
            mcw = wave_max(max_of(e));
            nw = ref_of(mcw);
            const float nref = nw == -INFINITY ? 0.f : nw;
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    e[j * EPV + k] = E::exp2_ref(e[j * EPV + k], nref);
                    sacc[k & 1] += (double)e[j * EPV + k];
                }
                __builtin_amdgcn_sched_barrier(0);                 // keep the working set to one vector at a time
            }
        }
        float ntw = -INFINITY;                                     // the reference this wave's Z_w is taken about
        bool tquads = MATRIX ? quads : MATRIX_T;             // the verifier row goes through the matrix cores
        double Zw = 0.0;
        if constexpr (LDS_NEXT) {
            // ---- T (these instances): the verifier row; its slots take the next centre row, which arrives during the rest
            if constexpr (DO_V) {
                take_row(buf);
                if (has_next) fetch_row(A.draft, next);
                __builtin_amdgcn_sched_barrier(0);
                verifier_mask(buf, quads ? kNoTokenWord : E::kNegInfWord);
                ntw = nw == -INFINITY ? 0.f : nw;
            }
            const int ol = opaque_tid() & 63;
            put_sum(sacc[0] + sacc[1], 5, ol);
            if constexpr (DO_V) put_sum(verifier_lane_sum(buf, ntw, quads), 6, ol);
            const double v = get_sums(ol);
            if (DO_Q && (ol & 7) == 0 && ol < 40) sm_q52[LDS_NEXT ? (done & 1) ^ 1 : 0][wave * NQ + (ol >> 3)] = v;   // (the row before's)
            auto of_group = [&](int g) {
                return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 8 * g), __builtin_amdgcn_readlane(__double2loint(v), 8 * g));
            };
            Sw = of_group(5);
            if constexpr (DO_V) {
                Zw = of_group(6);
                verifier_redo(buf, ntw, Zw, tquads);
            }
        } else {
            Sw = wave_sum(sacc[0] + sacc[1]);
        }

        // ---- the waves exchange the centre row's statistics ----------------------------------------------
        float (&sm_ref)[NW * 2] = sm_ref2[done & 1];
        double (&sm_S)[NW] = sm_S2[done & 1];
        float (&sm_nt)[NW] = sm_nt2[LDS_NEXT ? done & 1 : 0];
        double (&sm_Z)[NW] = sm_Z2[LDS_NEXT ? done & 1 : 0];
        double (&sm_q5)[NW * NQ] = sm_q52[0];                      // (LDS_NEXT: see put_sum)
        if (lane == 0) {
            sm_ref[wave * 2] = mcw; sm_ref[wave * 2 + 1] = nw;
            sm_S[wave] = Sw;
            if (DO_Q && wave == 0) sm_e0 = e[0];
            if constexpr (LDS_NEXT && DO_V) { sm_nt[wave] = ntw; sm_Z[wave] = Zw; }
        }
        row_barrier();
        // Combining the waves' results.  With eight waves or more every wave does it across its first lanes (lane
        // l < NW takes wave l; the other lanes of the DPP row repeat wave 0, which changes no maximum, and add
        // nothing); with four a short loop is as quick (measured).
        constexpr bool LANES = NW >= 8;
        const int ln = FORM_ANEW ? opaque_tid() & 63 : lane;
        const int src = ln < NW ? ln : 0;
        // (by_lanes: across the first lanes of the wave, which must all be active; else in a loop)
        auto combine_S = [&](auto by_lanes, float& mc, float& n, double& S) {
            if constexpr (decltype(by_lanes)::value) {
                // (n is the largest of the waves' references.  It is ref_of(mc) as well, but formed from mc it comes later and in a
                // vector register: one 1024-token row verified 5.45 -> 5.63 us, 36621 of them 109 -> 116, 65104 bf16 rows
                // quantified and verified with a radius tensor 529 -> 620)
                const float mc_l = sm_ref[src * 2], n_l = sm_ref[src * 2 + 1];
                mc = row16_max(mc_l); n = row16_max(n_l);
                S = row16_sum(ln < NW && n_l != -INFINITY ? sm_S[src] * pow2_of(n_l - n) : 0.0);
            } else {
                mc = sm_ref[0]; n = sm_ref[1];
#pragma unroll
                for (int w = 1; w < NW; ++w) {
                    mc = fmaxf(mc, sm_ref[w * 2]);
                    n = fmaxf(n, sm_ref[w * 2 + 1]);
                }
                S = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float rn = sm_ref[w * 2 + 1];
                    if (rn != -INFINITY) S += sm_S[w] * pow2_of(rn - n);
                }
            }
        };
        float mc, n;
        double S;                                                  // in units of 2^-n
        combine_S(std::integral_constant<bool, LANES>{}, mc, n, S);
        const float Sf = (float)S;                                 // for the accept test (see accept_quick)
        const double fw = nw == -INFINITY ? 0.0 : pow2_of(nw - n);     // this wave's e_i are 1/fw too large

        // ---- C: InterFuse sums in this wave's units, rescaled to row units by lane 0 of the wave ---------
        // Caps: S_l <= b / (1 - (1-b) x_max) and S_u >= a / (1 + (a-1) x_max) for the largest probability
        // x_max of the row, so below the host-computed bound on x_max both caps are inactive and the
        // cheaper width-only pass is exact.  Uniform over the workgroup.
        const double emax = (double)E::exp2_ref(mc, n);               // the row's largest e_i, in row units
        const bool capless = !A.normalize || (!RAD && emax <= A.capless_xmax * S);
        const bool split = emax > 0.5 * S;                         // some x_i above 1/2: 1 - x needs the two-float 1/S
        const bool flat = emax * (double)V <= 2.0 * S;             // largest probability <= 2 / V (see Shift)
        if constexpr (EARLY_NEXT) {
            __builtin_amdgcn_sched_barrier(0);
            if (has_next) load_row(buf, A.draft, next);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (EARLY_T) {
            // the verifier row goes in flight now, into the registers the centre row came in, and lands
            // during the interval pass
            __builtin_amdgcn_sched_barrier(0);
            load_row(buf, A.target, row);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (DO_Q) {
            // x_i = e_i fw / S: hand fuse_row the partition sum expressed in this wave's units
            // (fw is a power of two: the division is a change of exponent)
            const double Su = nw == -INFINITY ? 1.0 : ldexp(S, (int)fminf(n - nw, kFarUnits));   // S / fw
            // (the call's a, b and polynomial bound through opaque copies in scalar registers: what is derived from
            // them -- a - 1, 1 - b, the bound as a double -- is then formed here, an instruction each, instead of ahead
            // of the row loop, where it is kept in vector registers, or spilled, for all of it)
            double ra = A.a, rb = A.b;
            float wpx = A.wpoly_x;
            if constexpr (sizeof(T) == 2) asm volatile("" : "+s"(ra), "+s"(rb), "+s"(wpx));   // (fp32 instances: no gain, measured)
            // (by division in the bf16 instances of 1024 lanes, which spill: 1017 rows of 65536 tokens 168 -> 158 us)
            const FuseRow fr = TOP_INDEX ? fuse_row(Su, ra, rb) : fuse_row_inv(recip(Su), ra, rb);
            double q5[NQ];
            auto shift_of = [&](float eref, const FuseRow& r) {
                Shift k;
                k.kc = 0.f;
                if constexpr (RAD) {
                    if constexpr (WIDE) fuse_token_rad_wide<T>(eref, raw0, r, rm, k.kl, k.kw, k.kc);
                    else fuse_token_rad<T>(eref, raw0, r, rm, k.kl, k.kw);
                } else {
                    if constexpr (WIDE) fuse_token_wide(eref, r, k.kl, k.kw, k.kc);
                    else fuse_token<true>(eref, r, k.kl, k.kw);
                }
                return k;
            };
            // The common shift of a flat row (see Shift), 0 elsewhere.  A wave whose units are too far from the
            // row's (scalar radius) or from wave 0's (tensor radius) to form it takes its sums about 0, and its
            // lane 0 moves them to the common shift afterwards.
            bool near = false;
            Shift sh = {0.f, 0.f, 0.f};
            if (CIAR_RARE(HINTS, flat)) {
                if constexpr (RAD) {
                    const float up = sm_ref[1] - nw;               // e0 is 2^up times larger in this wave's units
                    near = fabsf(up) <= 64.f;                      // uniform over the wave; false for inf and nan
                    if (near) sh = shift_of(ldexpf(sm_e0, (int)up), fr);
                } else {
                    near = fw >= 0x1p-64;                          // uniform over the wave
                    if (near) sh = shift_of((float)(Su / (double)V), fr);
                }
            }
            // the width polynomial of this call's radius in this wave's units (x = e / S)
            WidthPoly wp = {0.f, 0.f, 0.f, 0.f, -1.f};
            if constexpr (!RAD && !WIDE) {
                const float is = -fr.nih, is2 = is * is;
                wp.d0 = A.wpoly[0] * is; wp.d1 = A.wpoly[1] * is2; wp.d2 = A.wpoly[2] * (is2 * is);
                wp.d3 = A.wpoly[3] * (is2 * is2);
                wp.ethr = wpx < 0.f || !ref_is_near(n) ? -1.f : (float)((double)wpx * Su);
                // uniform over the wave: scalar registers (an FMA reads one of them per issue, so d2 stays a vector)
                auto uniform = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
                wp.d0 = uniform(wp.d0); wp.d1 = uniform(wp.d1); wp.d3 = uniform(wp.d3); wp.ethr = uniform(wp.ethr);
            }
            double kq[3] = {(double)sh.kl, (double)sh.kw, (double)sh.kc};   // fp64 copy (the tiny path sets its own)
            const int base = slot_base(MATRIX && quads, MATRIX ? opaque_tid() : tid, EPV), step4 = slot_step(MATRIX && quads, EPV);
            bool tiny = false;
            if constexpr (NVEC == 1) tiny = V <= kTinyVocab;       // uniform
            if (CIAR_RARE(HINTS, tiny)) {
                if constexpr (NVEC == 1) {
                    if constexpr (RAD) {
                        __builtin_amdgcn_sched_barrier(0);
                        load_row(buf, A.radius, row);
                        E::zero_tail(buf[0], tid * EPV, V);
                    }
                    // all tokens sit in wave 0, whose lane 0 holds the first one
                    fuse_sums_tiny<T, EPV, RAD, WIDE>(e, buf[0], Su, A.a, A.b, A.kappa, A.rmax,
                                                      tid * EPV, V, q5, kq);
#pragma unroll
                    for (int i = 0; i < 5; ++i) q5[i] = wave_sum(q5[i]);
                }
            } else if constexpr (RAD) {
                // the raw radius row comes into the registers the centre row came in
                __builtin_amdgcn_sched_barrier(0);
                load_row(buf, A.radius, row);
                if (TOP_INDEX && split && mcw == mc) {
                    // (uniform over the wave: it holds the row's largest token; as for TopToken)
                    const float etop = E::exp2_ref(mcw, nw);
                    int at = -1;
#pragma unroll
                    for (int i = 0; i < EPT; ++i) at = e[i] == etop ? i : at;
                    if (at >= 0) sm_top[TOP_INDEX ? done : 0] = (at / EPV * THREADS + tid) * EPV + at % EPV;
                }
                if (partial) {
#pragma unroll
                    for (int j = 0; j < NVEC; ++j) E::zero_tail(buf[j], (j * THREADS + tid) * EPV, V);
                }
                TopToken top = {!TOP_INDEX && split && mcw == mc, false, uniform_f(E::exp2_ref(mcw, nw)), 0.f};
                if (rm.unit) fuse_sums_rad<T, THREADS, NVEC, WIDE, true>(e, buf, fr, rm, sh, V, tid, q5, top);
                else         fuse_sums_rad<T, THREADS, NVEC, WIDE, false>(e, buf, fr, rm, sh, V, tid, q5, top);
                if (top.found) sm_rtop[TOP_INDEX ? 0 : done] = top.raw;            // (one lane of the workgroup), for finish_row
#pragma unroll
                for (int i = 0; i < 5; ++i) q5[i] = wave_sum(q5[i]);
            } else if constexpr (WIDE) {
                fuse_sums_wide<THREADS, NVEC, EPV>(e, fr, sh, V, base, step4, q5);
#pragma unroll
                for (int i = 0; i < 5; ++i) q5[i] = wave_sum(q5[i]);
            } else if (CIAR_USUAL(HINT_CAPS, capless)) {
                if (partial)    fuse_sums<THREADS, NVEC, EPV, true, true, true>(e, fr, wp, sh, V, base, step4, q5);
                else if (CIAR_RARE(HINTS, split)) fuse_sums<THREADS, NVEC, EPV, true, true, false>(e, fr, wp, sh, V, base, step4, q5);
                else            fuse_sums<THREADS, NVEC, EPV, true, false, false>(e, fr, wp, sh, V, base, step4, q5);
                if constexpr (!LDS_NEXT) {
                    q5[1] = wave_sum(q5[1]);
                    q5[3] = wave_sum(q5[3]);
                }
            } else {
                // (Sixteen vectors of bf16: only flat rows have a shift, and without one a slot past the row's end adds nothing by itself.  The
                // masks are more than the registers hold there: ten sums read back from scratch for every vector.  us, tiles of eight
                // vectors / masks on every ragged row / on flat ones, rows with one token of nearly all the mass: 4099 x 26001 255 / 381 / 185, 4099 x
                // 13001 144 / 203 / 101, 256 x 13000 26.8 / 34.9 / 23.0, 8 x 26000 30.2 / 39.1 / 23.4.)
                const bool masked = partial && (!(LDS_NEXT && NVEC == 16) || flat);
                if (masked) fuse_sums<THREADS, NVEC, EPV, false, true, true, FULL>(e, fr, wp, sh, V, base, step4, q5);
                else        fuse_sums<THREADS, NVEC, EPV, false, true, false>(e, fr, wp, sh, V, base, step4, q5);
                if constexpr (!LDS_NEXT) {
#pragma unroll
                    for (int i = 0; i < 5; ++i) q5[i] = wave_sum(q5[i]);
                }
            }
            if constexpr (WIDE) {
                q5[5] = wave_sum(q5[5]);
                q5[6] = wave_sum(q5[6]);
                q5[7] = (double)wave_max((float)q5[7]);
            }
            if constexpr (LDS_NEXT) {
                if (CIAR_RARE(HINTS, flat && !near)) {             // (uniform over the wave) the wave's sums, as from its lane 0
#pragma unroll
                    for (int i = 0; i < 5; ++i) {
                        q5[i] = wave_sum(q5[i]);
                        if (lane != 0) q5[i] = 0.0;
                    }
                }
            }
            if (LDS_NEXT || lane == 0) {
                // to row units (the complements are plain numbers: nothing to rescale)
                double ku = fw;
                const double f2 = fw * fw;
                q5[0] *= fw; q5[1] *= fw; q5[2] *= f2; q5[3] *= f2; q5[4] *= f2;
                // (the lane asked for only where it has to be: as a further term of the branch's condition, even a constant one, it made
                // the compiler keep the tiny rows' constants otherwise, and fused bf16 calls of 256 vectors with a radius tensor lost 9 %)
                bool move = flat && !near && !tiny;
                if constexpr (LDS_NEXT) move = move && lane == 0;
                if (CIAR_RARE(HINTS, move)) {
                    // Rare: this wave's sums are about 0.  Form the common shift the long way round, in row units
                    // (scalar radius) or in wave 0's (tensor radius), and move the sums to it:  with c = 0 - K and
                    // n tokens,  sum (d - K) = s1 + n c,  sum (d - K)^2 = s2 + 2 c s1 + n c^2,  likewise the cross
                    // moment.
                    double fw0 = 1.0;
                    Shift k0;
                    if constexpr (RAD) {
                        fw0 = pow2_of(sm_ref[1] - n);
                        k0 = shift_of(sm_e0, fuse_row(S / fw0, ra, rb));
                    } else {
                        k0 = shift_of((float)(S / (double)V), fuse_row(S, ra, rb));
                    }
                    kq[0] = (double)k0.kl * fw0; kq[1] = (double)k0.kw * fw0; kq[2] = (double)k0.kc;
                    ku = 1.0;
                    const double cl = -kq[0], cw = -kq[1], cc = -kq[2];
                    int cnt = 0;                                   // tokens of the row in this wave
                    // (from an opaque copy of the wave's index: the count does not change from row to row, and hoisted
                    // out of the row loop it is kept in registers, or spilled, for all of it)
                    int wv = wave;
                    asm volatile("" : "+v"(wv));
#pragma unroll
                    for (int j = 0; j < NVEC; ++j) cnt += min(max(V - (j * THREADS + wv * 64) * EPV, 0), 64 * EPV);
                    const double nn = (double)cnt;
                    q5[4] += cl * q5[1] + cw * (q5[0] + nn * cl);
                    q5[2] += cl * (2.0 * q5[0] + nn * cl);
                    q5[3] += cw * (2.0 * q5[1] + nn * cw);
                    q5[0] += nn * cl;
                    q5[1] += nn * cw;
                    if constexpr (WIDE) {
                        q5[6] += cc * (2.0 * q5[5] + nn * cc);
                        q5[5] += nn * cc;
                    }
                }
                if constexpr (LDS_NEXT) {
                    const int ol = opaque_tid() & 63;
                    put_sum(q5[1], 1, ol);
                    put_sum(q5[3], 3, ol);
                    if (CIAR_RARE(HINT_CAPS, !capless)) { put_sum(q5[0], 0, ol); put_sum(q5[2], 2, ol); put_sum(q5[4], 4, ol); }
                } else {
#pragma unroll
                    for (int i = 0; i < NQ; ++i) sm_q5[wave * NQ + i] = q5[i];
                }
                if (wave == 0 && lane == 0) { sm_k[0] = kq[0] * ku; sm_k[1] = kq[1] * ku; sm_k[2] = kq[2]; }
            }
        }

        // ---- T: verifier row statistics, per wave -----------------------------------------------------------
        if constexpr (DO_V && !LDS_NEXT) {
            if constexpr (!EARLY_T) {
                // no registers to spare next to the interval pass: the verifier row is fetched only now
                __builtin_amdgcn_sched_barrier(0);
                load_row(buf, A.target, row);
            }
            verifier_stats(buf, nw, ntw, Zw, tquads);
            if (lane == 0) { sm_nt[wave] = ntw; sm_Z[wave] = Zw; }
        }
        // The next centre row goes in flight before the barrier and thread 0's bookkeeping -- except where this
        // kernel makes the draws: there both rows stay in the registers until the accept test has been decided (below).
        if constexpr (!EARLY_NEXT && !KEEP_E && !LDS_NEXT) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (DO_V) {
                if (has_next) load_row(buf, A.draft, next);
            } else {
                load_row(buf, A.draft, has_next ? next : row, has_next);
            }
        }

        if constexpr (!LDS_NEXT) __syncthreads();

        // ---- verification of the drafted token, in every wave alike (Algorithm 1, "Cloud verification") ----------
        // Z and its reference over the waves; the accept test; on a rejection the draw from (q - p)+ by inverse CDF
        // in token order, from the registers: e[] still holds the centre row's exponentials, buf the verifier row.
        // Z and its reference over the waves, exactly (fp64): wanted by the lane that writes the row up and by a draw
        // (by_lanes: across the first lanes of the wave, which must all be active; else in a loop)
        auto combine_Z = [&](auto by_lanes, float& nt, double& Z) {
            nt = -INFINITY;
            Z = 0.0;                                               // in units of 2^-nt
            if constexpr (decltype(by_lanes)::value) {
                const float nt_l = sm_nt[src];
                nt = row16_max(nt_l);
                Z = row16_sum(ln < NW && nt_l != -INFINITY ? sm_Z[src] * pow2_of(nt_l - nt) : 0.0);
            } else {
#pragma unroll
                for (int w = 0; w < NW; ++w) nt = fmaxf(nt, sm_nt[w]);
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float rt = sm_nt[w];
                    if (rt != -INFINITY) Z += sm_Z[w] * pow2_of(rt - nt);
                }
            }
        };
        // (Where resample_kernel makes the draws nothing in this loop depends on the accept test: the lane that
        // finishes the row evaluates it, in fp64.)
        if constexpr (DO_V && KEEP_E) {
            // for the accept test in fp32 a float Z does (every wave evaluates it: kept short)
            float ntq = -INFINITY, Zq = 0.f;
            if constexpr (LANES) {
                const float nt_l = sm_nt[src];
                ntq = row16_max(nt_l);
                Zq = row16_sum_f(ln < NW && nt_l != -INFINITY ? ldexpf((float)sm_Z[src], (int)fmaxf(nt_l - ntq, -200.f)) : 0.f);
            } else {
#pragma unroll
                for (int w = 0; w < NW; ++w) ntq = fmaxf(ntq, sm_nt[w]);
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    const float rt = sm_nt[w];
                    if (rt != -INFINITY) Zq += ldexpf((float)sm_Z[w], (int)fmaxf(rt - ntq, -200.f));
                }
            }
            const float cx = sm_fx[done][0], tx = sm_fx[done][2], ua = sm_fx[done][3];
            // 1 = accepted, 0 = rejected, -1 = too close to call in fp32: then the draw is made as well, and the
            // lane that finishes the row decides in fp64 whether it counts (about one row in a few thousand)
            const int verdict = accept_quick(cx, tx, ua, n, ntq, Sf, Zq);
            if (tid == 0) sm_close[done] = (uint8_t)(verdict < 0);
            if (CIAR_USUAL(HINTS, verdict > 0)) {
                if (tid == 0) sm_draw[done] = -1;
            } else {
                // p_i = e_i pfac, q_i = 2^(t_i log2e - ntw) qfac, res_i = max(0, q_i - p_i) rounded to fp32: every
                // partial sum below is a sum of those floats, so that the totals of the pieces and the running sum
                // inside the piece that holds u R are sums of the same numbers.  (Not of the same roundings: a lane adds its
                // tokens in fp32 before the lanes are added in fp64, and with transposed slots the totals' lanes hold other tokens of their
                // quad than the running sum's.  The two differ by about 1e-7 of a lane's mass; a u R that falls into the difference
                // at a piece's end draws that piece's last token with mass, see lastpos.)
                // (the lane index goes through an empty asm, so that nothing of this branch is computed ahead of the
                // row loop and kept in registers, or spilled, for all of it)
                int dt = tid;
                asm volatile("" : "+v"(dt));
                const int dlane = dt & 63, dwave = dt >> 6;
                // the row's scalars again, from the exchange slots (nothing of them is kept in registers for this
                // branch; the slots are this row's until the next row's second barrier)
                float dmc, n, nt;
                double S, Z;
                combine_S(std::integral_constant<bool, LANES>{}, dmc, n, S);
                combine_Z(std::integral_constant<bool, LANES>{}, nt, Z);
                const float nw = sm_ref[dwave * 2 + 1], ntw = sm_nt[dwave];
                const double fw = nw == -INFINITY ? 0.0 : pow2_of(nw - n);
                // q - p in fp32, as resample_kernel forms it: the product e / S is rounded once (6e-8 of p, below the ~1e-7
                // of p and of q that the fp32 exponentials carry anyway) and the FMA takes the difference from the exact
                // product of the verifier's exponential and 1 / Z
                const float pfac = LDS_NEXT ? (float)(fw * recip(S)) : (float)(fw / S);
                float ntref = ntw == -INFINITY ? 0.f : ntw;
                // (opaque to the optimiser, like e below: it would otherwise keep the streaming passes' conversions
                // and exponentials of every token alive for this branch, in registers the hot path does not have)
                asm volatile("" : "+v"(ntref));
                const double qscale = ntw == -INFINITY ? 0.0 : pow2_of(ntw - nt);
                const float qfac = LDS_NEXT && Z > 0x1p-900 && Z < 0x1p900 ? (float)(qscale * recip(Z)) : (float)(qscale / Z);
                // (a centre row in transposed slots: the verifier row's tokens likewise, or, where that row may not go through
                // the matrix cores, the centre row's put in order)
                auto residuals = [&](int j, float (&r)[EPV]) {
                    if constexpr (MATRIX) {
                        if (quads && tquads) {
                            float tz[EPV];
                            bf16_scaled(buf[j], bf16_scale(dt), tz);
#pragma unroll
                            for (int k = 0; k < EPV; ++k) {
                                float ek = e[j * EPV + k];
                                asm volatile("" : "+v"(ek));
                                r[k] = fmaxf(fmaf(exp2_scaled(tz[k], ntref), qfac, -(ek * pfac)), 0.f);
                            }
                            return;
                        }
                    }
                    float tv[EPV], ev[EPV];
                    E::unpack(buf[j], tv);
#pragma unroll
                    for (int k = 0; k < EPV; ++k) ev[k] = e[j * EPV + k];
                    if constexpr (MATRIX) {
                        if (quads) {
#pragma unroll
                            for (int g = 0; g < EPV; g += 4) quad_transpose(ev[g], ev[g + 1], ev[g + 2], ev[g + 3], dt);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < EPV; ++k) {
                        float ek = ev[k];
                        asm volatile("" : "+v"(ek));
                        r[k] = fmaxf(fmaf(E::exp2_ref(tv[k], ntref), qfac, -(ek * pfac)), 0.f);
                    }
                };
                // Piece totals.  Eight vectors per lane: the eight lane sums are reduced over the wave together -- two DPP
                // steps leave every quad's sum in its lanes, the quad leaders put it into LDS vector by vector, then lane l
                // takes two of the 16 quad sums of vector l / 8 and three butterfly steps over its eight lanes finish all
                // eight totals (a DPP reduction of one double over a wave is ~36 instructions: eight of them were a third
                // of a draw).  Fewer vectors: one reduction each.
                if constexpr (LDS_NEXT) {
                    // Sixteen vectors: the lanes' sums first, one vector's products ahead of the next one's arithmetic and no branch
                    // in between (with two waves per SIMD nobody else fills the gaps of a chain per vector); then four vectors at a
                    // time through LDS, lane l adding those of lanes 4 (l % 16) ... + 3 of vector l / 16 and a reduction over 16
                    // lanes finishing all four.
                    auto sum_of = [](const float (&r)[EPV]) {
                        const float a = (r[0] + r[1]) + (r[2] + r[3]);
                        return EPV == 4 ? a : a + ((r[4 % EPV] + r[5 % EPV]) + (r[6 % EPV] + r[7 % EPV]));
                    };
                    float* const slots = reinterpret_cast<float*>(&sm_quad[dwave][0][0]);   // [4][64]
                    constexpr int GROUPS = (NVEC + 3) / 4;
                    double part[GROUPS];
                    float sums[4] = {0.f, 0.f, 0.f, 0.f};
                    auto four = [&](int g) {
                        // (LDS operations of a wave complete in order)
#pragma unroll
                        for (int v = 0; v < 4; ++v) slots[v * 64 + dlane] = sums[v];
                        const u32x4 w = *reinterpret_cast<const u32x4*>(slots + 4 * dlane);
                        part[g] = ((double)bits_f(w.x) + (double)bits_f(w.y)) + ((double)bits_f(w.z) + (double)bits_f(w.w));
                    };
                    if (CIAR_USUAL(HINTS, quads && tquads)) {
                        const Bf16Scale bs = bf16_scale(dt);
                        float tz[2][EPV];
                        bf16_scaled(buf[0], bs, tz[0]);
#pragma unroll
                        for (int j = 0; j < NVEC; ++j) {
                            if (j + 1 < NVEC) bf16_scaled(buf[j + 1], bs, tz[(j + 1) & 1]);
                            float r[EPV];
#pragma unroll
                            for (int k = 0; k < EPV; ++k) {
                                r[k] = fmaxf(fmaf(exp2_scaled(tz[j & 1][k], ntref), qfac, -(e[j * EPV + k] * pfac)), 0.f);
                            }
                            sums[j & 3] = sum_of(r);
                            if ((j & 3) == 3 || j == NVEC - 1) four(j / 4);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < NVEC; ++j) {
                            float r[EPV];
                            residuals(j, r);
                            sums[j & 3] = sum_of(r);
                            if ((j & 3) == 3 || j == NVEC - 1) four(j / 4);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g) part[g] = dpp_add<kRowShr1, 0xf>(part[g]);
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g) part[g] = dpp_add<kRowShr2, 0xf>(part[g]);
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g) part[g] = dpp_add<kRowShr4, 0xf>(part[g]);
#pragma unroll
                    for (int g = 0; g < GROUPS; ++g) part[g] = dpp_add<kRowShr8, 0xf>(part[g]);
                    if ((dlane & 15) == 15) {
#pragma unroll
                        for (int g = 0; g < GROUPS; ++g)
                            if (4 * g + (dlane >> 4) < NVEC) sm_tab[(4 * g + (dlane >> 4)) * NW + dwave] = part[g];
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < NVEC; ++j) {
                        float sj = 0.f;
                        if (j * CHUNK < V) {                       // uniform: the vector holds tokens
                            float r[EPV];
                            residuals(j, r);
#pragma unroll
                            for (int k = 0; k < EPV; ++k) sj += r[k];
                        }
                        if constexpr (NVEC == 8) {
                            double q = (double)sj;
                            q = dpp_add<0xB1, 0xf>(q);             // lane ^ 1  (quad_perm 1,0,3,2)
                            q = dpp_add<0x4E, 0xf>(q);             // lane ^ 2  (quad_perm 2,3,0,1)
                            if ((dlane & 3) == 0) sm_quad[dwave][j][dlane >> 2] = q;
                        } else {
                            const double ws = wave_sum((double)sj);
                            if (dlane == 0) sm_tab[j * NW + dwave] = ws;
                        }
                    }
                    if constexpr (NVEC == 8) {
                        // (the wave reads what its own lanes have written: LDS operations of a wave complete in order)
                        const double* pr = &sm_quad[dwave][dlane >> 3][2 * (dlane & 7)];
                        double t2 = pr[0] + pr[1];
                        t2 = dpp_add<0xB1, 0xf>(t2);
                        t2 = dpp_add<0x4E, 0xf>(t2);
                        t2 = dpp_add<0x141, 0xf>(t2);              // the other quad of the eight (row_half_mirror)
                        if ((dlane & 7) == 0) sm_tab[(dlane >> 3) * NW + dwave] = t2;
                    }
                }
                row_barrier();
                // every wave locates the piece that holds u R: lane l takes piece l (and l + 64), an inclusive scan
                // over the lanes gives the running sums in token order, a ballot the first one above u R
                constexpr int PER = (NT + 63) / 64;
                double tot[PER], run[PER], carry = 0.0;
                auto lane_value = [&](double v, int from) {
                    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), from),
                                            __builtin_amdgcn_readlane(__double2loint(v), from));
                };
#pragma unroll
                for (int p = 0; p < PER; ++p) {
                    const int idx = p * 64 + dlane;
                    tot[p] = idx < NT ? sm_tab[idx] : 0.0;
                    run[p] = wave_scan(tot[p]) + carry;
                    carry = lane_value(run[p], 63);
                }
                const double R = carry;
                const float ur = sm_ur[done];
                if (CIAR_USUAL(HINT_DRAW, R > 0.0)) {
                    const double thr = (double)ur * R;
                    int istar = -1;
                    double before = 0.0;
                    double prev_end = 0.0;                         // running sum at the end of the part before
#pragma unroll
                    for (int p = 0; p < PER; ++p) {
                        const unsigned long long cross = __ballot(p * 64 + dlane < NT && run[p] > thr);
                        if (istar < 0 && cross) {
                            const int l = __builtin_amdgcn_readfirstlane(__ffsll((long long)cross) - 1);
                            istar = p * 64 + l;
                            before = l > 0 ? lane_value(run[p], l - 1) : prev_end;
                        }
                        prev_end = lane_value(run[p], 63);
                    }
                    if (CIAR_RARE(HINT_DRAW, istar < 0)) {                               // unreachable for u < 1; keeps the draw valid
#pragma unroll
                        for (int p = 0; p < PER; ++p) {
                            const unsigned long long live = __ballot(p * 64 + dlane < NT && tot[p] > 0.0);
                            if (live) istar = p * 64 + __builtin_amdgcn_readfirstlane(63 - __clzll((long long)live));
                        }
                        before = R;
                    }
                    const int wstar = istar % NW, jstar = istar / NW;
                    if (dwave == wstar) {
                        int cand = INT_MAX, lastpos = -1;
                        // smallest token of the piece whose inclusive running sum exceeds u R; tokens without
                        // residual mass cannot be drawn; lastpos covers a crossing lost to rounding at its end
                        auto scan_piece = [&](int j, float (&r)[EPV]) {
                            if constexpr (MATRIX) {
                                if (quads && tquads) {
#pragma unroll
                                    for (int g = 0; g < EPV; g += 4) quad_transpose(r[g], r[g + 1], r[g + 2], r[g + 3], dt);
                                }
                            }
                            float s = 0.f;
#pragma unroll
                            for (int k = 0; k < EPV; ++k) s += r[k];
                            const double incl = wave_scan((double)s);
                            double cum = before + (incl - (double)s);
                            const int base = (j * THREADS + dt) * EPV;
                            auto search = [&](int& above, int& last) {
#pragma unroll
                                for (int k = 0; k < EPV; ++k) {
                                    cum += (double)r[k];
                                    if (r[k] > 0.f) {
                                        last = base + k;
                                        if (cum > thr && above == INT_MAX) above = base + k;
                                    }
                                }
                            };
                            // (local: selections, not branches.  1024 lanes have no registers for them: fp32 4328 x 31744 226.5 us in place,
                            // 229.4 local, with 8 B of scratch)
                            if constexpr (THREADS < 1024) {
                                int above = INT_MAX, last = -1;
                                search(above, last);
                                cand = above;
                                lastpos = last;
                            } else {
                                search(cand, lastpos);
                            }
                        };
                        // (j == jstar is uniform; the register arrays keep constant indices.  The scan once behind the choice of the vector:
                        // sixteen copies of it are half a draw's instructions to fetch; of one or two the calls of few rows lose 5 % so.)
                        float chosen[EPV];
#pragma unroll
                        for (int j = 0; j < NVEC; ++j) {
                            if (j == jstar) {
                                if constexpr (LDS_NEXT) {
                                    residuals(j, chosen);
                                } else {
                                    float r[EPV];
                                    residuals(j, r);
                                    scan_piece(j, r);
                                }
                            }
                        }
                        if constexpr (LDS_NEXT) scan_piece(jstar, chosen);
                        cand = wave_min_i(cand);
                        lastpos = wave_max_i(lastpos);
                        if (dlane == 0) {
                            const int id = cand != INT_MAX ? cand : lastpos;
                            sm_draw[done] = id < 0 ? 0 : id;
                        }
                    }
                } else {
                    // every residual rounded to zero (q == p to working precision): the draw degenerates to the
                    // lowest-index arg-max of q, which is that of the verifier logits; practically never taken
                    float mt = -INFINITY;
#pragma unroll
                    for (int j = 0; j < NVEC; ++j) {
                        float tv[EPV];
                        E::unpack(buf[j], tv);
#pragma unroll
                        for (int k = 0; k < EPV; ++k) mt = fmaxf(mt, tv[k]);
                    }
                    mt = wave_max(mt);
                    if (dlane == 0) sm_auxf[dwave] = mt;
                    row_barrier();
#pragma unroll
                    for (int w = 0; w < NW; ++w) mt = fmaxf(mt, sm_auxf[w]);
                    int ci = INT_MAX;
#pragma unroll
                    for (int j = 0; j < NVEC; ++j) {
                        float tv[EPV];
                        E::unpack(buf[j], tv);
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            const int tok = (j * THREADS + dt) * EPV + k;
                            if (tv[k] == mt && tok < V) ci = min(ci, tok);
                        }
                    }
                    ci = wave_min_i(ci);
                    if (dlane == 0) sm_auxi[dwave] = ci;
                    row_barrier();
                    if (dt == 0) {
                        int c0 = sm_auxi[0];
#pragma unroll
                        for (int w = 1; w < NW; ++w) c0 = min(c0, sm_auxi[w]);
                        sm_draw[done] = c0 == INT_MAX ? 0 : c0;
                    }
                }
            }
            // both rows are spent: the next centre row goes in flight
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!LDS_NEXT) {
                if (has_next) load_row(buf, A.draft, next);
            }
        }

        // ---- wave 0 leaves the row's ten numbers for the finishing -------------------------------------------------
        // Sixteen waves: their results are combined across the first lanes as above; fewer: by lane 0 in a loop
        // (as quick, measured).  Handing this job from wave to wave in turn measured slower.
        if constexpr (LDS_NEXT) {
            // (the interval sums follow behind the next row's barrier)
            if (wave == 0) {
                float nt = -INFINITY;
                double Z = 0.0;
                if constexpr (DO_V) combine_Z(std::integral_constant<bool, LANES>{}, nt, Z);
                if (lane == 0) {
                    RowStats& st = sm_rows[done];
                    st.S = S; st.Z = Z; st.n = n; st.nt = nt; st.mc = mc;
                    float mode = capless ? kSumsWidthOnly : kSumsFull;
                    if (DO_Q && A.precise_flat && flat && V > kTinyVocab) mode += kSumsFlatPending;
                    st.kl = DO_Q ? sm_k[0] : 0.0; st.kw = DO_Q ? sm_k[1] : 0.0;
                    st.mode = mode;
                    if constexpr (!DO_Q) {
#pragma unroll
                        for (int i = 0; i < 5; ++i) st.q[i] = 0.0;
                    }
                }
                if (DO_Q && done > 0) park_sums_of(done - 1, (done & 1) ^ 1);
            }
        }
        if (!LDS_NEXT && wave == 0 && (NW >= 16 || lane == 0)) {
            float mc, n, nt = -INFINITY;
            double S, Z = 0.0;
            combine_S(std::integral_constant<bool, (NW >= 16)>{}, mc, n, S);
            if constexpr (DO_V) combine_Z(std::integral_constant<bool, (NW >= 16)>{}, nt, Z);
            double t[NQ];
#pragma unroll
            for (int i = 0; i < NQ; ++i) t[i] = 0.0;
            double K[3] = {0.0, 0.0, 0.0};
            if constexpr (DO_Q) { K[0] = sm_k[0]; K[1] = sm_k[1]; K[2] = sm_k[2]; }
            // the waves' interval sums are about one common shift (wave 0 left it in row units): they simply add
            if constexpr (DO_Q) {
                if constexpr (NW >= 16) {
#pragma unroll
                    for (int i = 0; i < NQ; ++i) {
                        const double mine = ln < NW ? sm_q5[src * NQ + i] : 0.0;
                        t[i] = i == 7 ? (double)row16_max((float)mine) : row16_sum(mine);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < NQ; ++i) {
#pragma unroll
                        for (int w = 0; w < NW; ++w)
                            t[i] = i == 7 ? fmax(t[i], sm_q5[w * NQ + i]) : t[i] + sm_q5[w * NQ + i];
                    }
                }
            }
            if (lane == 0) {
                RowStats stv;
                RowStats* const st = &stv;
                st->S = S; st->Z = Z; st->n = n; st->nt = nt; st->mc = mc;
                float mode = (capless && !WIDE) ? kSumsWidthOnly : kSumsFull;
                if constexpr (WIDE && DO_Q) {
                    // every width above 1/2 and both caps inactive: the finishing reads the complement sums
                    if (t[7] < kComplementBelow) {
                        const RowScore rs = finish_score(t, S, kSumsFull, A, K[0], K[1]);
                        if (rs.alpha_l == 1.0 && rs.alpha_u == 1.0) {
                            t[1] = t[5]; t[3] = t[6]; K[1] = K[2];
                            mode = kSumsComplement;
                        }
                    }
                }
                // a flat row of a call whose widths are not small: the fp64 pass behind this kernel redoes its sums
                if (DO_Q && A.precise_flat && flat && V > kTinyVocab) mode += kSumsFlatPending;
                st->kl = K[0]; st->kw = K[1];
                st->mode = mode;
#pragma unroll
                for (int i = 0; i < 5; ++i) st->q[i] = t[i];
                // with finishing the statistics stay in LDS until the batch is finished
                if (finish) sm_rows[done] = stv;
                else A.stats[row] = stv;
            }
        }

        if (!has_next) break;
        row = next;
        // Wave priority by progress (set here for the next row; the first row runs at priority 3): the workgroups of a compute unit are served oldest first, so the one that was
        // dispatched first runs at full speed and the others on what it leaves (a timeline of the benchmark launch: the
        // first workgroup of every compute unit took 7.5 us per row and ended at 39 us, the second 12 us per row and ended
        // at 49 us, alone on its compute unit for the last 10 us).  A workgroup therefore runs the first quarter of its
        // rows at priority 3, the second at 2, ...: whoever is behind is served first, and the workgroups of a compute
        // unit end together (benchmark 55.6 -> 52.8 us per step, workload 4 347 -> 328 us, workload 3 276 -> 257 us).
        // Not where a compute unit holds one workgroup only (1024 lanes), and not for a single row.
        if constexpr (THREADS < 1024) {
            if (cnt > 1) {
                // (uniform; floor(4 done / cnt) without a division: compares and shifts on scalar registers)
                if ((done + 1) < ((cnt + 3) >> 2)) __builtin_amdgcn_s_setprio(3);
                else if ((done + 1) < ((cnt + 1) >> 1)) __builtin_amdgcn_s_setprio(2);
                else if ((done + 1) < ((3 * cnt + 3) >> 2)) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
            }
        }
    }
    if constexpr (LDS_NEXT && DO_Q) {
        const int ol = opaque_tid() & 63;
        const double v = get_sums(ol);
        if ((ol & 7) == 0 && ol < 40) sm_q52[LDS_NEXT ? (cnt - 1) & 1 : 0][wave * NQ + (ol >> 3)] = v;
        __syncthreads();
        if (wave == 0) park_sums_of(cnt - 1, (cnt - 1) & 1);
    }
    if (finish) finish_batch(L0, cnt);
}

// ---- dispatch ---------------------------------------------------------------------------------------------

template <typename T, int THREADS, int NVEC, bool DO_Q, bool DO_V, bool RAD, bool WIDE = false>
hipError_t launch_stream_kernel(const RowArgs& a, StreamLaunch& L)
{
    if (a.V < full_vectors<T, THREADS, NVEC, DO_V, RAD, WIDE>() * THREADS * Elt<T>::kPerVec) return hipErrorInvalidValue;
    // One wave of resident workgroups, each walking over its pieces of rows with stride gridDim.x.
    const int64_t resident = (int64_t)workgroups_per_unit<T, THREADS, NVEC, DO_Q, DO_V, RAD, WIDE>() * L.units;
    const int64_t N = a.N;
    constexpr int ROWS = rows_per_wg<T, THREADS, NVEC, DO_V, RAD, WIDE>();   // (at most so many rows per workgroup)
    const int64_t grid1 = whole_rounds(N, ROWS, resident), max1 = (N + grid1 - 1) / grid1;
    StreamPlan& p = L.plan;
    p.unit = 1;
    p.grid = (unsigned)grid1;
    p.rows_per_wg = (int)max1;
    p.windows_inline = false;
    if (DO_V && (a.accept_len || a.resampled_id) && a.window >= 1 && a.window <= ROWS) {
        // Whole windows per workgroup, so that the kernel writes the window outputs as well, unless that would leave
        // the busiest workgroup with noticeably more rows than a row-by-row split (few windows on many compute units)
        const int64_t K = a.window, units = (N + K - 1) / K;
        const int64_t gridk = whole_rounds(units, ROWS / K, resident), maxk = (units + gridk - 1) / gridk * K;
        if (maxk <= max1 + max1 / 8) {
            p.unit = (int)K;
            p.grid = (unsigned)gridk;
            p.rows_per_wg = (int)maxk;
            p.windows_inline = true;
        }
    }
    p.can_finish = DO_V || L.finish_rows;
    p.draws_inline = draws_in_stream<T, THREADS, NVEC, DO_V, RAD, WIDE>();
    // Windows that span workgroups: where this kernel knows every row's draw it can still write the window outputs,
    // from the lane that finishes a window's last row (one 64-bit word per window in the workspace, see window_arrive).
    // (Its rows arrive one after another: with one row to a workgroup all of a window at once, and long windows take longer so than a
    // launch of window_kernel.  us, counted / window_kernel, verified bf16 rows of 8629 tokens: 123 rows, windows of 16 16.3 / 15.4, of 31
    // 22.0 / 14.6, of 100 71 / 15; 1000 rows, of 16 21.3 / 21.9, of 31 27.3 / 22.3; 9000 rows, nine to a workgroup, of 31 89.4 / 93.4,
    // of 100 135 / 94.  A call with fewer rows than a window has only those to count: windows of 31, fused fp32 rows of 16244 tokens
    // 1 row 12.2 / 13.7, 10 rows 15.9 / 17.2, 16 rows 18.4 / 17.3; bf16 of 7614 tokens 10 rows 13.0 / 13.8, 12 rows 14.0 / 13.8, 16 rows
    // 15.5 / 13.8; verified fp32 10 rows 12.8 / 12.8.)
    p.windows_counted = p.draws_inline && a.win_words && (a.accept_len || a.resampled_id) && !p.windows_inline && a.window >= 2 &&
                        (a.window <= (p.rows_per_wg > 3 ? kMaxCountedWindow : 16) || N <= 10);

    if (!L.launch) return hipSuccess;
    RowArgs b = a;
    b.finish = p.can_finish ? 1 : 0;
    b.unit = p.unit;
    b.win_count = p.windows_counted ? a.win_words : nullptr;
    auto kernel = &stream_kernel<T, THREADS, NVEC, DO_Q, DO_V, RAD, WIDE, false>;
    if constexpr (!WIDE && (DO_V || !RAD) && NVEC != 12) {                       // (quantify-only calls with a radius tensor: V <= 64 comes here)
        if (b.V == NVEC * THREADS * Elt<T>::kPerVec) kernel = &stream_kernel<T, THREADS, NVEC, DO_Q, DO_V, RAD, WIDE, true>;
    }
    constexpr unsigned lds = next_by_lds<T, THREADS, NVEC, DO_V, RAD, WIDE>() ? THREADS * NVEC * 16u : 0u;
    if constexpr (lds > 32 * 1024 - 1) {
        // with the static arrays above the default limit: raised once per device and instance
        static std::mutex guard;
        static bool raised[2][64] = {};
        const int whole = kernel == &stream_kernel<T, THREADS, NVEC, DO_Q, DO_V, RAD, WIDE, false> ? 0 : 1;
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        std::lock_guard<std::mutex> lock(guard);
        if (!raised[whole][dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            raised[whole][dev] = true;
        }
    }
    if (L.ev_start && L.ev_stop)
        hipExtLaunchKernelGGL(kernel, dim3(p.grid), dim3(THREADS), lds, L.stream, L.ev_start, L.ev_stop, 0, b);
    else
        hipLaunchKernelGGL(kernel, dim3(p.grid), dim3(THREADS), lds, L.stream, b);
    return hipGetLastError();
}

}  // namespace
}  // namespace ciar
