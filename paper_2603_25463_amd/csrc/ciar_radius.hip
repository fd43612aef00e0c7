// gfx950 quantifier for calls with a radius tensor and no verifier row (Sec. 3.2.3: r = Softplus of the Interval Head's radius
// half): ciar_quantify in tensor mode, every head of Voting, the consumer of ciar_interhead_quantify.
//
// Two rows per position, the second of which (the raw radius) is wanted only once the partition sum of the first is known.
// Per row, in a workgroup that walks over its rows:
//   1. centre row: per-wave maximum, e_i = 2^(c_i log2e - n_w) in registers, S_w;  -- barrier: (max, S_w) --
//   2. radius row, vector by vector: p^l_i and p^u_i - p^l_i from e_i, S and the token's own a_i - 1; five sums.
// Both rows come through the same slots of LDS (global_load_lds: no register is held while a row is on its way): when the centre
// row has moved to registers its slots are requested full of the radius row, which arrives during step 1, and every slot
// that step 2 has read is requested full of the next centre row, which arrives during the rest of step 2.  A lane reads back
// only slots that its own wave has requested, so the hand-over is the wave's own count of outstanding loads.  128 bytes of a
// row per lane (32 fp32 or 64 bf16 tokens) at four waves per SIMD: what a row costs a wave whatever its length (reductions,
// exchange, constants: ~300 instructions) is spread over as many tokens as the registers hold.
// What the streaming kernel did for such calls before: the radius row requested into registers behind the barrier (its trip to
// memory exposed, two thirds of the time of a row), bf16 rows with 76-250 B of scratch per lane, a second launch for flat
// rows and a third for the vote.
//
// A row's scalars are parked in LDS; after the workgroup's last row a lane per row turns them into the outputs.  Rows whose
// widths (or whose complements) agree to better than kCrowded says and flat rows of calls whose widths are not small
// (needs_flat_pass) are swept again in fp64 before that is written.
#include "ciar_device.h"

#include <hip/hip_ext.h>
#include <mutex>

namespace ciar {
namespace {

// 16-byte vectors of a row per lane.  (bf16 rows with complement sums: 32 tokens; with 64 those instances spill 136 to 208 bytes,
// which is left for the rows above 32768 tokens.)
constexpr int kRadVecs = 8, kRadVecsWide16 = 4;
// Rows whose Sigma is below three thousandths of the mean width are swept again in fp64.  (What the fp32 rounding of the widths --
// 1e-7 of each, but alike for like tokens -- leaves in a Sigma at that line: 2e-6 to 7e-6 of it, 256 to 16384 tokens, clamps
// of 0.5 to 4; 1e-5 to 4e-5 at a third of it.  At a hundredth it would be 5e-7 to 2e-6, but there rows of an untrained head pay
// for the sweep in calls with a small clamp: 762 x 16384 fp32, radius_max 2, 209 us against 24.5.)
constexpr double kCrowded = 1e-5;
constexpr double kCapGuard = 1e-5;     // how far from its cap a sum of bounds taken in fp32 (good to ~1e-6) has to be to settle it
// The estimate of sum p - p^l from which a wave expects inactive caps (they are from 0.01 on).  On rows of radii around 0.018 the estimates of
// 64 tokens scatter by 0.0025: at 0.015 one wave in ten expects the worse, at 0.0125 one in a hundred.
constexpr float kExpectInactive = 0.0125f;
template <int THREADS> constexpr int radius_rows() { return THREADS >= 512 ? 128 : THREADS / 4; }   // most rows of a workgroup

template <bool WIDE> struct RadiusRow { double S, q[WIDE ? 7 : 5]; float n, mc, raw_top, big; };   // see RowStats, finish_row

// The five sums of a row in fp64 from the logits, about the first token's values, by the whole workgroup; red: 6 doubles per wave.
template <typename T, int THREADS>
__device__ void radius_row_fp64(const RowArgs& A, int64_t row, double (*red)[64], RowStats& st)
{
    constexpr int NW = THREADS / 64;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const T* crow = static_cast<const T*>(A.draft) + row_offset(A, row);
    const T* rrow = static_cast<const T*>(A.radius) + row_offset(A, row);
    const double mc = (double)st.mc;
    auto total = [&](double v) {
        v = wave_sum(v);
        __syncthreads();                                           // the slots may still be read from the last use
        if (lane == 0) red[wave][0] = v;
        __syncthreads();
        return row16_sum(lane < NW ? red[lane < NW ? lane : 0][0] : 0.0);
    };
    double s = 0.0;
    for (int i = tid; i < A.V; i += THREADS) s += exp((double)load_logit(crow, i) - mc);   // masked token: exp(-inf) = 0
    const double invS = 1.0 / total(s);
    auto token = [&](int i, double& pl, double& w) {
        const double x = exp((double)load_logit(crow, i) - mc) * invS;
        const double r = radius_of((double)load_logit(rrow, i), A.kappa, A.rmax);
        const double a = exp(r), b = exp(-r), om = 1.0 - x, dl = b + (1.0 - b) * om, du = 1.0 + (a - 1.0) * x;
        pl = b * x / dl;
        w = (a - b) * x * om / (du * dl);
    };
    double kl, kw;
    token(0, kl, kw);                                              // every lane forms the same shift
    double q[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int i = tid; i < A.V; i += THREADS) {
        double pl, w;
        token(i, pl, w);
        pl -= kl; w -= kw;
        q[0] += pl; q[1] += w;
        q[2] = fma(pl, pl, q[2]); q[3] = fma(w, w, q[3]); q[4] = fma(pl, w, q[4]);
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) st.q[i] = total(q[i]);
    st.kl = kl; st.kw = kw;
    st.mode = kSumsDirect;
}

// The five sums of a row in the units of its logits' reference, by the whole workgroup from the logits: the token arithmetic of
// radius_kernel, for a row whose caps turned out not to be inactive.
template <typename T, int THREADS, bool UNIT>
__device__ void radius_row_full(const RowArgs& A, int64_t row, double (*red)[64], RowStats& st)
{
    using E = Elt<T>;
    constexpr int EPV = E::kPerVec, NW = THREADS / 64;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6, V = A.V;
    const gbytes crow = (gbytes)(static_cast<const T*>(A.draft) + row_offset(A, row));
    const gbytes rrow = (gbytes)(static_cast<const T*>(A.radius) + row_offset(A, row));
    const float n = st.n == -INFINITY ? 0.f : st.n, kappa = (float)A.kappa, rmax = (float)A.rmax;
    const FuseRow fr = fuse_row_inv(recip(st.S), A.a, A.b);
    double q[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int j = tid; j * EPV < V; j += THREADS) {
        u32x4 cb = *(gvec)(crow + (uint32_t)j * 16u), rb = *(gvec)(rrow + (uint32_t)j * 16u);
        E::mask_tail(cb, j * EPV, V);
        E::zero_tail(rb, j * EPV, V);
        float cv[EPV], rv[EPV];
        E::unpack(cb, cv);
        E::unpack(rb, rv);
#pragma unroll
        for (int k = 0; k < EPV; ++k) {
            float pl, w;
            fuse_token_rad<T, UNIT>(E::exp2_ref(cv[k], n), rv[k], fr, kappa, rmax, A.am1_max, pl, w);
            const double dl = (double)pl, dw = (double)w;
            q[0] += dl; q[1] += dw;
            q[2] = fma(dl, dl, q[2]); q[3] = fma(dw, dw, q[3]); q[4] = fma(dl, dw, q[4]);
        }
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) q[i] = wave_sum(q[i]);
    __syncthreads();                                               // the slots may still be read from the last use
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < 5; ++i) red[wave][i] = q[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 5; ++i) st.q[i] = row16_sum(lane < NW ? red[lane < NW ? lane : 0][i] : 0.0);
    st.kl = 0.0; st.kw = 0.0;
    st.mode = kSumsFull;
}

// ---- what radius_kernel and radius_lean_kernel have in common ------------------------------------------------------------

// The lane's index, asked for anew wherever it is used, through an empty asm: no LDS address formed from it is held in registers, or
// spilled, through the row loop -- and a reload would wait for the row in flight.
__device__ __forceinline__ int my_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

template <typename T>
__device__ __forceinline__ gbytes radius_row_base(const RowArgs& A, int H, const void* rows, uint32_t pos, int h)
{
    const int64_t off = H > 1 ? (int64_t)h * A.head_stride + (int64_t)pos * A.stride : row_offset(A, pos);
    const uint64_t b = (uint64_t)(static_cast<const T*>(rows) + off);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return (gbytes)(((uint64_t)hi << 32) | lo);
}

// Vector j of a row goes in flight (lane l of a wave lands 16 l bytes behind the address the wave names); lanes past the end of
// the row fetch its last vector.
template <int THREADS>
__device__ __forceinline__ void fetch_vector(gbytes base, u32x4* slots, int j, int wave, int tid, uint32_t last_off)
{
    using lds_ptr = __attribute__((address_space(3))) void*;
    using glb_ptr = const __attribute__((address_space(1))) void*;
    __builtin_amdgcn_global_load_lds((glb_ptr)(base + min((uint32_t)(j * THREADS + tid) * 16u, last_off)),
                                     (lds_ptr)(slots + j * THREADS + wave * 64), 16, 0, kNonTemporal);
}

// The sum over eight lanes, in each of them: lane ^ 1, lane ^ 2, the other quad.
__device__ __forceinline__ double sum_of_eight(double v)
{
    v = dpp_add<0xB1, 0xf>(v);
    v = dpp_add<0x4E, 0xf>(v);
    return dpp_add<0x141, 0xf>(v);
}

// One wave: a row's sums over the workgroup's waves.
template <int NW, int NQ>
__device__ __forceinline__ void park_sums(const double (&tot)[NW][NQ], double* q, int lane)
{
    const int grp = lane >> 3, part = lane & 7;
    double v = 0.0;
    if (grp < NQ) {
        if (part < NW) v = tot[part][grp];
        if (NW > 8) v += tot[part + (NW > 8 ? 8 : 0)][grp];
    }
    v = sum_of_eight(v);
    if (grp < NQ && part == 0) q[grp] = v;
}

// Wave priority by progress: whoever of the workgroups of a compute unit is behind is served first.
__device__ __forceinline__ void priority_by_progress(int done, int count)
{
    if (done < (count + 3) >> 2) __builtin_amdgcn_s_setprio(3);
    else if (done < (count + 1) >> 1) __builtin_amdgcn_s_setprio(2);
    else if (done < (3 * count + 3) >> 2) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// A lane finishes a row, see finish_row, with its arg-max token (ARGMAX) or the drafted one.  The flag is left for the vote, which
// counts the flags as written.
template <typename T, bool ARGMAX, typename Again>
__device__ __forceinline__ bool finish_radius_row(const RowArgs& A, int64_t r, int argmax, const RowStats& st, float raw_top,
                                                  uint8_t* flag, Again again)
{
    const int64_t off = row_offset(A, r);
    int xid = ARGMAX ? argmax : A.ids ? A.ids[ids_index(A, r)] : 0;
    xid = xid < 0 ? 0 : (xid >= A.V ? A.V - 1 : xid);
    const float cx = load_logit(static_cast<const T*>(A.draft) + off, xid);
    const float rawx = load_logit(static_cast<const T*>(A.radius) + off, xid);
    if (finish_row<T, true>(A, r, st, cx, 0.f, rawx, 0.f, true, false, raw_top, flag, again)) return true;
    A.stats[r] = st;
    return false;
}

// The strict majority of the workgroup's positions' flags.
__device__ __forceinline__ void vote_of_positions(const uint8_t* flags, int H, int mine, uint32_t step, uint8_t* __restrict__ votes)
{
    __syncthreads();
    const int t = my_tid();
    if (t < mine) {
        int yes = 0;
        for (int i = 0; i < H; ++i) yes += flags[t * H + i];
        votes[blockIdx.x + (int64_t)t * step] = (uint8_t)(2 * yes > H);
    }
}

// ---- the kernels -----------------------------------------------------------------------------------------------------------

// A.N rows: H > 1: [H, P], H heads of P = A.head_rows positions, the H rows of a position one after another in one workgroup,
// which can then vote; H = 1: P = A.N rows dealt singly, of one head or of several (see row_offset).
// ARGMAX = no drafted ids: every row reports its arg-max token.  votes: [P] flags by strict majority, or null.
// WIDE = radii at which the widths can crowd against 1 (wide_radius): rows of which every width is above 1/2 take their Omega and
// Sigma from the sums of the complements 1 - width (fuse_token_rad_wide), which are formed where they may be wanted: a width
// above 1/2 has (a + 1) x > 1, and a wave of which one lane's first token has not spares itself the rest.
template <typename T, int THREADS, int NVEC, bool UNIT, bool ARGMAX, bool WIDE>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(4)))
void radius_kernel(const RowArgs A, const int H, uint8_t* __restrict__ votes)
{
    using E = Elt<T>;
    constexpr int EPV = E::kPerVec, EPT = NVEC * EPV, NW = THREADS / 64, ROWS = radius_rows<THREADS>();
    constexpr int CHUNK = THREADS * EPV;                           // tokens of one vector of every lane
    extern __shared__ u32x4 sm_next[];                             // [NVEC][THREADS]: the row in flight
    // exchange slots of a row: written before its barrier, read behind it; rows alternate between two sets
    // per wave: largest logit; bf16: and the reference n_w.  (Formed again from the largest logits by every wave, 2048 x 4096 bf16 19.5 us, 8
    // rows 8.7, so 18.8 and 8.4; fp32 rows lose up to 2 % so.)
    constexpr bool REFS = sizeof(T) == 2;
    __shared__ float sm_ref[2][NW][REFS ? 2 : 1];
    constexpr int NQ = WIDE ? 7 : 5;                               // sums of a row
    __shared__ double sm_S[2][NW], sm_tot[2][NW][NQ];
    __shared__ double sm_red[NW][64];                              // per wave: [the sums of the row before, S_w][eight groups of lanes]
    __shared__ float sm_big[WIDE ? 2 : 1][NW];                     // largest complement
    // (LDS is what the places on a compute unit are counted by: a slot per wave and parked row instead of this pair costs the
    // 128-lane instances one of eight, 58333 x 3000 fp32 270 -> 350 us)
    __shared__ int sm_pi[2][ARGMAX ? NW : 1];
    // parked rows
    __shared__ RadiusRow<WIDE> pk[ROWS];
    __shared__ int pk_id[ARGMAX ? ROWS : 1];
    __shared__ uint8_t pk_fp64[ROWS], pk_flag[ROWS];

    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int V = A.V;
    const int nch = (V + CHUNK - 1) / CHUNK;                       // vectors of a lane that hold tokens at all
    const int last_vec = (V + EPV - 1) / EPV - 1;
    const uint32_t P = (uint32_t)(H > 1 ? A.head_rows : A.N), step = gridDim.x;
    const float kappa = uniform_f((float)A.kappa), rmax = uniform_f((float)A.rmax), am1_max = A.am1_max;
    // this workgroup's rows: H of each of its positions blockIdx.x, blockIdx.x + step, ...
    const uint32_t mine = blockIdx.x < P ? (P - blockIdx.x + step - 1u) / step : 0u;
    const int count = (int)mine * H;                               // <= ROWS: the launcher sizes the grid accordingly
    if (count == 0) return;

    auto row_base = [&](const void* rows, uint32_t pos, int h) { return radius_row_base<T>(A, H, rows, pos, h); };
    const uint32_t last_off = (uint32_t)last_vec * 16u;
    auto fetch = [&](gbytes base, int j, int tid) {
        if (j < nch) fetch_vector<THREADS>(base, sm_next, j, wave, tid, last_off);   // uniform
    };
    // wave 0: a row's sums over the waves, parked
    auto park = [&](int at, int p) {
        const int lane = my_tid() & 63;
        park_sums(sm_tot[p], pk[at].q, lane);
        if constexpr (WIDE) {
            const float big = row16_max(lane < NW ? sm_big[p][lane < NW ? lane : 0] : 0.f);
            if (lane == 0) pk[at].big = big;
        }
    };
    // the sums of a wave reduced together: every lane's value -> groups of eight lanes (three DPP steps) -> LDS
    auto put = [&](double v, int which, int lane) {
        v = sum_of_eight(v);
        if ((lane & 7) == 0) sm_red[wave][which * 8 + (lane >> 3)] = v;
    };
    auto get = [&](int lane) { return sum_of_eight(sm_red[wave][lane < 8 * (NQ + 1) ? lane : 0]); };   // lanes 8 q ...: quantity q

    uint32_t pos = blockIdx.x;
    int h = 0;
    {
        const gbytes base = row_base(A.draft, pos, h);
        const int tid = my_tid();
#pragma unroll
        for (int j = 0; j < NVEC; ++j) fetch(base, j, tid);
    }
    if constexpr (THREADS < 1024) {
        if (count > 1) __builtin_amdgcn_s_setprio(3);
    }
    for (int done = 0;; ++done) {
        const int p = done & 1;
        const int tid = my_tid(), lane = tid & 63;
        const bool has_next = done + 1 < count;                    // uniform
        // ---- 1: the centre row ------------------------------------------------------------------------------------------
        float e[EPT];
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        {
            u32x4 buf[NVEC];
#pragma unroll
            for (int j = 0; j < NVEC; ++j) buf[j] = sm_next[j * THREADS + tid];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            const gbytes base = row_base(A.radius, pos, h);
#pragma unroll
            for (int j = 0; j < NVEC; ++j) fetch(base, j, tid);
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
                if ((j + 1) * CHUNK > V) E::mask_tail(buf[j], (j * THREADS + tid) * EPV, V);      // uniform
                E::unpack(buf[j], &e[j * EPV]);
            }
        }
        const float mw = wave_max(max_of(e)), nw = ref_of(mw), nref = nw == -INFINITY ? 0.f : nw;
        if constexpr (ARGMAX) {
            int at = INT_MAX;
#pragma unroll
            for (int i = EPT - 1; i >= 0; --i)
                if (e[i] == mw) at = (i / EPV * THREADS + tid) * EPV + i % EPV;
            at = wave_min_i(at);
            if (lane == 0) sm_pi[p][wave] = at;
        }
        double Sl = 0.0;
#pragma unroll
        for (int j = 0; j < NVEC; ++j) {
            if (j < nch) {
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    e[j * EPV + k] = Elt<T>::exp2_ref(e[j * EPV + k], nref);
                    Sl += (double)e[j * EPV + k];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        put(Sl, NQ, lane);
        {
            const double v = get(lane);
            const int grp = lane >> 3;
            if ((lane & 7) == 0) {
                if (grp < NQ) { if (done > 0) sm_tot[p ^ 1][wave][grp] = v; }
                else if (grp == NQ) sm_S[p][wave] = v;
            }
            if (lane == 0) {
                sm_ref[p][wave][0] = mw;
                if constexpr (REFS) sm_ref[p][wave][1] = nw;
            }
        }
        lds_barrier();
        if (wave == 0 && done > 0) park(done - 1, p ^ 1);
        const int src = lane < NW ? lane : 0;
        const float m_l = sm_ref[p][src][0], mc = row16_max(m_l);
        const float n_l = REFS ? sm_ref[p][src][REFS ? 1 : 0] : ref_of(m_l), n = REFS ? row16_max(n_l) : ref_of(mc);
        const double S = row16_sum(lane < NW && n_l != -INFINITY ? sm_S[p][src] * pow2_of(n_l - n) : 0.0);
        if constexpr (ARGMAX) {
            if (wave == 0) {                                       // the lowest index of the waves that hold the maximum
                const int best = wave_min_i(lane < NW && m_l == mc ? sm_pi[p][src] : INT_MAX);
                if (lane == 0) pk_id[done] = best == INT_MAX ? 0 : best;
            }
        }
        if (tid == 0) { pk[done].S = S; pk[done].n = n; pk[done].mc = mc; }
        const double fw = nw == -INFINITY ? 0.0 : pow2_of(nw - n);                         // this wave's e_i are 1 / fw too large
        const double Su = nw == -INFINITY ? 1.0 : ldexp(S, (int)fminf(n - nw, kFarUnits));   // S in this wave's units
        const bool top = (double)Elt<T>::exp2_ref(mc, n == -INFINITY ? 0.f : n) > 0.5 * S;         // uniform over the workgroup
        FuseRow fr;
        {
            const double inv = recip(Su);
            const float nih = (float)-inv;
            fr = {0.f, uniform_f(nih), uniform_f((float)(-inv - (double)nih)), 0.f, 0.f};
        }
        // ---- 2: the radius row; its slots take the next centre row as they are read ---------------------------------------
        uint32_t npos = pos;
        int nh = h;
        if (has_next) {
            if (++nh == H) { nh = 0; npos += step; }
        }
        const gbytes next = row_base(A.draft, npos, nh);
        double q[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) q[i] = 0.0;
        // A row with a token above 1/2: its raw radius is parked for finish_row by the lane that has it, in the wave with the row's
        // largest token.  (No other token has its e: two of them would be all of S.)
        const bool search = top && mw == mc;                       // uniform over the wave
        const float etop = uniform_f(Elt<T>::exp2_ref(mw, nref));
        float raw_top = 0.f;
        bool found = false;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bool complements = false;                                  // uniform over the wave
        float big = INFINITY;                                      // largest complement of this lane
        constexpr int GROUP = WIDE && sizeof(T) == 2 ? 2 : 4;      // vectors taken at a time
#pragma unroll
        for (int g = 0; g < NVEC; g += GROUP) {
            u32x4 rb[GROUP];
#pragma unroll
            for (int u = 0; u < GROUP; ++u) rb[u] = sm_next[(g + u) * THREADS + tid];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (has_next) {
#pragma unroll
                for (int u = 0; u < GROUP; ++u) fetch(next, g + u, tid);
            }
#pragma unroll
            for (int u = 0; u < GROUP; ++u) {
                const int j = g + u;
                if (j < nch) {                                     // uniform: the vectors hold tokens
                    if ((j + 1) * CHUNK > V) E::zero_tail(rb[u], (j * THREADS + tid) * EPV, V);
                    float rv[EPV];
                    E::unpack(rb[u], rv);
                    if (WIDE && j == 0) {
                        const float am1 = radius_am1<T, UNIT>(rv[0], kappa, rmax, am1_max);
                        complements = __builtin_amdgcn_ballot_w64(tid * EPV < V && !(-(am1 + 2.0f) * e[0] * fr.nih > 1.0f)) == 0;
                        if (complements) big = 0.f;
                    }
                    if (WIDE && complements) {
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            float pl, w, ec;
                            fuse_token_rad_wide<T, UNIT>(e[j * EPV + k], rv[k], fr, kappa, rmax, am1_max, pl, w, ec);
                            if ((j * THREADS + tid) * EPV + k < V) {   // (past the row's end ec is not 0)
                                const double dc = (double)ec;
                                q[NQ - 2] += dc; q[NQ - 1] = fma(dc, dc, q[NQ - 1]);
                                big = fmaxf(big, ec);
                            }
                            const double dl = (double)pl, dw = (double)w;
                            q[0] += dl; q[1] += dw;
                            q[2] = fma(dl, dl, q[2]); q[3] = fma(dw, dw, q[3]); q[4] = fma(dl, dw, q[4]);
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            float pl, w;                               // (a slot past the row's end holds e = 0: both are 0)
                            fuse_token_rad<T, UNIT>(e[j * EPV + k], rv[k], fr, kappa, rmax, am1_max, pl, w);
                            const double dl = (double)pl, dw = (double)w;
                            q[0] += dl; q[1] += dw;
                            q[2] = fma(dl, dl, q[2]); q[3] = fma(dw, dw, q[3]); q[4] = fma(dl, dw, q[4]);
                        }
                    }
                    if (search) {
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            const bool is = e[j * EPV + k] == etop;
                            raw_top = is ? rv[k] : raw_top;
                            found = found || is;
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (found) pk[done].raw_top = raw_top;                     // (one lane of the workgroup)
        {
            const double f2 = fw * fw;                             // to row units
            put(q[0] * fw, 0, lane); put(q[1] * fw, 1, lane);
            put(q[2] * f2, 2, lane); put(q[3] * f2, 3, lane); put(q[4] * f2, 4, lane);
            if constexpr (WIDE) {
                if (complements) {                                 // (else the two sums are whatever their slots hold, and not used)
                    put(q[NQ - 2], NQ - 2, lane); put(q[NQ - 1], NQ - 1, lane);     // (plain numbers: nothing to rescale)
                    big = wave_max(big);
                }
                if (lane == 0) sm_big[p][wave] = big;
            }
        }
        if (!has_next) break;
        pos = npos; h = nh;
        if constexpr (THREADS < 1024) priority_by_progress(done + 1, count);
    }
    {
        const int lane = my_tid() & 63;
        const double v = get(lane);
        if ((lane & 7) == 0 && lane < 8 * NQ) sm_tot[(count - 1) & 1][wave][lane >> 3] = v;
    }
    __syncthreads();
    if (wave == 0) park(count - 1, (count - 1) & 1);
    __syncthreads();
    // ---- a lane per row ---------------------------------------------------------------------------------------------------
    auto stats_of = [&](int at) {
        RowStats st;
        st.S = pk[at].S; st.Z = 0.0; st.n = pk[at].n; st.nt = 0.f; st.mc = pk[at].mc;
#pragma unroll
        for (int i = 0; i < 5; ++i) st.q[i] = pk[at].q[i];
        st.kl = 0.0; st.kw = 0.0; st.mode = kSumsFull;
        if constexpr (WIDE) {
            if (pk[at].big < (float)kComplementBelow) {            // every width above 1/2
                const RowScore rs = finish_score(st.q, st.S, kSumsFull, A, 0.0, 0.0);
                if (rs.alpha_l == 1.0 && rs.alpha_u == 1.0) { st.q[1] = pk[at].q[NQ - 2]; st.q[3] = pk[at].q[NQ - 1]; st.mode = kSumsComplement; }
            }
        }
        return st;
    };
    auto row_of = [&](int at) { return (int64_t)(at % H) * P + blockIdx.x + (int64_t)(at / H) * step; };
    auto finish = [&](int at, const RowStats& st, auto again) {
        return finish_radius_row<T, ARGMAX>(A, row_of(at), pk_id[ARGMAX ? at : 0], st, pk[at].raw_top, &pk_flag[at], again);
    };
    {
        const int t = my_tid();
        // (the statistics alone, for the Ensemble's second sweep, which looks after its own flat rows)
        const bool outputs = A.p_lo || A.p_mid || A.p_hi || A.omega || A.sigma || A.score || A.flags;
        if (t < count && !outputs) {
            pk_fp64[t] = 0;
            A.stats[row_of(t)] = stats_of(t);
        } else if (t < count) {
            const RowStats st = stats_of(t);
            const double etop = (double)Elt<T>::exp2_ref(st.mc, st.n == -INFINITY ? 0.f : st.n);
            pk_fp64[t] = (uint8_t)finish(t, st, [&](const RowScore& rs) {
                const double Vd = (double)V, mean = (WIDE && st.mode == kSumsComplement ? Vd - rs.omega : rs.omega) / Vd;
                return !(rs.sigma * rs.sigma >= kCrowded * mean * mean) || (A.precise_flat && etop * Vd <= 2.0 * st.S);
            });
        }
    }
    __syncthreads();
    for (int at = 0; at < count; ++at) {
        if (!pk_fp64[at]) continue;                                // uniform
        RowStats st = stats_of(at);
        radius_row_fp64<T, THREADS>(A, row_of(at), sm_red, st);
        if (my_tid() == 0) finish(at, st, NeverAgain{});
    }
    if (votes) vote_of_positions(pk_flag, H, (int)mine, step, votes);
}

// The same for calls whose rows follow one another (see launch_radius_tile): where a row's caps are expected to be inactive a wave
// takes the sums of the widths alone (`lean` below), and bf16 rows go through the matrix cores.  2048 x 16384, three heads, bf16
// 112.4 -> 102.5 us; 1531 x 12345 fp32 36.3 -> 35.2.
template <typename T, int THREADS, int NVEC, bool UNIT, bool ARGMAX>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(4)))
void radius_lean_kernel(const RowArgs A, const int H, uint8_t* __restrict__ votes)
{
    using E = Elt<T>;
    constexpr int EPV = E::kPerVec, EPT = NVEC * EPV, NW = THREADS / 64, ROWS = radius_rows<THREADS>();
    constexpr int CHUNK = THREADS * EPV;                           // tokens of one vector of every lane
    constexpr bool MATRIX = sizeof(T) == 2;                        // rows go through the matrix cores (see bf16_scaled)
    constexpr bool SCALED = MATRIX && UNIT;                        // the radius row's tokens are taken times kBf16Scale
    extern __shared__ u32x4 sm_next[];                             // [NVEC][THREADS]: the row in flight
    // exchange slots of a row: written before its barrier, read behind it; rows alternate between two sets
    __shared__ float sm_ref[2][NW];
    constexpr int NQ = 5;                                          // sums of a row
    __shared__ double sm_S[2][NW], sm_tot[2][NW][NQ];
    __shared__ double sm_red[NW][64];                              // per wave: [the sums of the row before, S_w][eight groups of lanes]
    // (LDS is what the places on a compute unit are counted by: a slot per wave and parked row instead of this pair costs the
    // 128-lane instances one of eight, 58333 x 3000 fp32 270 -> 350 us)
    __shared__ int sm_pi[2][ARGMAX ? NW : 1];
    // parked rows
    __shared__ RadiusRow<false> pk[ROWS];
    __shared__ int pk_id[ARGMAX ? ROWS : 1];
    __shared__ uint8_t pk_fp64[ROWS], pk_flag[ROWS];

    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int V = A.V;
    const int nch = (V + CHUNK - 1) / CHUNK;                       // vectors of a lane that hold tokens at all
    const int last_vec = (V + EPV - 1) / EPV - 1;
    const uint32_t P = (uint32_t)(H > 1 ? A.head_rows : A.N), step = gridDim.x;
    const float kappa = uniform_f((float)A.kappa), rmax = uniform_f((float)A.rmax), am1_max = A.am1_max;
    // this workgroup's rows: H of each of its positions blockIdx.x, blockIdx.x + step, ...
    const uint32_t mine = blockIdx.x < P ? (P - blockIdx.x + step - 1u) / step : 0u;
    const int count = (int)mine * H;                               // <= ROWS: the launcher sizes the grid accordingly
    if (count == 0) return;

    auto row_base = [&](const void* rows, uint32_t pos, int h) { return radius_row_base<T>(A, H, rows, pos, h); };
    const uint32_t last_off = (uint32_t)last_vec * 16u;
    auto fetch = [&](gbytes base, int j, int tid) {
        if (j < nch) fetch_vector<THREADS>(base, sm_next, j, wave, tid, last_off);   // uniform
    };
    // wave 0: a row's sums over the waves, parked
    auto park = [&](int at, int p) {
        const int lane = my_tid() & 63;
        park_sums(sm_tot[p], pk[at].q, lane);
    };
    // the sums of a wave reduced together: every lane's value -> groups of eight lanes (three DPP steps) -> LDS
    auto put = [&](double v, int which, int lane) {
        v = sum_of_eight(v);
        if ((lane & 7) == 0) sm_red[wave][which * 8 + (lane >> 3)] = v;
    };
    auto get = [&](int lane) { return sum_of_eight(sm_red[wave][lane < 8 * (NQ + 1) ? lane : 0]); };   // lanes 8 q ...: quantity q

    uint32_t pos = blockIdx.x;
    int h = 0;
    {
        const gbytes base = row_base(A.draft, pos, h);
        const int tid = my_tid();
#pragma unroll
        for (int j = 0; j < NVEC; ++j) fetch(base, j, tid);
    }
    if constexpr (THREADS < 1024) {
        if (count > 1) __builtin_amdgcn_s_setprio(3);
    }
    for (int done = 0;; ++done) {
        const int p = done & 1;
        const int tid = my_tid(), lane = tid & 63;
        const bool has_next = done + 1 < count;                    // uniform
        // ---- 1: the centre row ------------------------------------------------------------------------------------------
        float e[EPT];
        float mw, nw;
        bool quads = false;                                        // the slots of e[] are transposed (uniform over the wave)
        double Sl = 0.0;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        {
            u32x4 buf[NVEC];
#pragma unroll
            for (int j = 0; j < NVEC; ++j) buf[j] = sm_next[j * THREADS + tid];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            const gbytes base = row_base(A.radius, pos, h);
#pragma unroll
            for (int j = 0; j < NVEC; ++j) fetch(base, j, tid);
            if constexpr (MATRIX) {
#pragma unroll
                for (int j = 0; j < NVEC; ++j)
                    if ((j + 1) * CHUNK > V) E::mask_tail(buf[j], (j * THREADS + tid) * EPV, V, kNoTokenWord);   // uniform
                mw = wave_top(top_words(buf), quads);
            }
            if (MATRIX && __builtin_expect(quads, true)) {
                nw = ref_of(mw);
                if constexpr (ARGMAX) {
                    int at = INT_MAX;
#pragma unroll
                    for (int j = NVEC - 1; j >= 0; --j) {
                        float v[EPV];
                        E::unpack(buf[j], v);
#pragma unroll
                        for (int k = EPV - 1; k >= 0; --k)
                            if (v[k] == mw) at = j * EPV + k;
                    }
                    at = wave_min_i(at == INT_MAX ? INT_MAX : (at / EPV * THREADS + tid) * EPV + at % EPV);
                    if (lane == 0) sm_pi[p][wave] = at;
                    __builtin_amdgcn_sched_barrier(0);
                }
                const Bf16Scale bs = bf16_scale(tid);
                bf16_scaled(buf[0], bs, &e[0]);
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    if (j + 1 < NVEC) bf16_scaled(buf[j + 1], bs, &e[(j + 1) * EPV]);   // (the matrix cores one vector ahead)
                    if (j < nch) {
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            e[j * EPV + k] = exp2_scaled(e[j * EPV + k], nw);
                            Sl += (double)e[j * EPV + k];
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    if ((j + 1) * CHUNK > V) E::mask_tail(buf[j], (j * THREADS + tid) * EPV, V);      // uniform
                    E::unpack(buf[j], &e[j * EPV]);
                }
                mw = wave_max(max_of(e));
                nw = ref_of(mw);
                const float nref = nw == -INFINITY ? 0.f : nw;
                if constexpr (ARGMAX) {
                    int at = INT_MAX;
#pragma unroll
                    for (int i = EPT - 1; i >= 0; --i)
                        if (e[i] == mw) at = i;
                    at = wave_min_i(at == INT_MAX ? INT_MAX : (at / EPV * THREADS + tid) * EPV + at % EPV);
                    if (lane == 0) sm_pi[p][wave] = at;
                }
#pragma unroll
                for (int j = 0; j < NVEC; ++j) {
                    if (j < nch) {
#pragma unroll
                        for (int k = 0; k < EPV; ++k) {
                            e[j * EPV + k] = Elt<T>::exp2_ref(e[j * EPV + k], nref);
                            Sl += (double)e[j * EPV + k];
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        put(Sl, NQ, lane);
        {
            const double v = get(lane);
            const int grp = lane >> 3;
            if ((lane & 7) == 0) {
                if (grp < NQ) { if (done > 0) sm_tot[p ^ 1][wave][grp] = v; }
                else if (grp == NQ) sm_S[p][wave] = v;
            }
            if (lane == 0) sm_ref[p][wave] = mw;
        }
        lds_barrier();
        if (wave == 0 && done > 0) park(done - 1, p ^ 1);
        const int src = lane < NW ? lane : 0;
        const float m_l = sm_ref[p][src], n_l = ref_of(m_l), mc = row16_max(m_l), n = ref_of(mc);
        const double S = row16_sum(lane < NW && n_l != -INFINITY ? sm_S[p][src] * pow2_of(n_l - n) : 0.0);
        if constexpr (ARGMAX) {
            if (wave == 0) {                                       // the lowest index of the waves that hold the maximum
                const int best = wave_min_i(lane < NW && m_l == mc ? sm_pi[p][src] : INT_MAX);
                if (lane == 0) pk_id[done] = best == INT_MAX ? 0 : best;
            }
        }
        if (tid == 0) { pk[done].S = S; pk[done].n = n; pk[done].mc = mc; }
        const double fw = nw == -INFINITY ? 0.0 : pow2_of(nw - n);                         // this wave's e_i are 1 / fw too large
        const double Su = nw == -INFINITY ? 1.0 : ldexp(S, (int)fminf(n - nw, kFarUnits));   // S in this wave's units
        const bool top = (double)Elt<T>::exp2_ref(mc, n == -INFINITY ? 0.f : n) > 0.5 * S;         // uniform over the workgroup
        FuseRow fr;
        {
            const double inv = recip(Su);
            const float nih = (float)-inv;
            fr = {0.f, uniform_f(nih), uniform_f((float)(-inv - (double)nih)), 0.f, 0.f};
        }
        // ---- 2: the radius row; its slots take the next centre row as they are read ---------------------------------------
        uint32_t npos = pos;
        int nh = h;
        if (has_next) {
            if (++nh == H) { nh = 0; npos += step; }
        }
        const gbytes next = row_base(A.draft, npos, nh);
        double q[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) q[i] = 0.0;
        // A row with a token above 1/2: its raw radius is parked for finish_row by the lane that has it, in the wave with the row's
        // largest token.  (No other token has its e: two of them would be all of S.)
        const bool search = top && mw == mc;                       // uniform over the wave
        const float etop = uniform_f(Elt<T>::exp2_ref(mw, nw == -INFINITY ? 0.f : nw));
        float raw_top = 0.f;
        bool found = false;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // Where the caps are inactive -- they are on almost every row -- Omega and Sigma want the sums of the widths alone (see
        // kSumsWidthOnly).  Whether they are is known when the row is summed, so a wave that expects it takes those two in
        // fp64 and sum p^l in fp32, which tells (kCapGuard), and marks the row by a sum that is no number; a row that was
        // expected wrong is taken again (radius_row_full).  21 instead of 27 issues per token.
        // The expectation: the caps are inactive where sum p^u - p and sum p - p^l, whose tokens with small p have p (1 - b) as their
        // common lower bound, are above a hundredth.  The wave estimates that sum from its lanes' first tokens, none of which counts
        // for more than a quarter of what it takes: a likely token says nothing of the others (kExpectInactive).
        // (Weighed by p, for a row that is taken again costs as much once more: where the likely tokens have small radii and the others
        // large ones 2048 x 12345 fp32 took 88 us when the radii alone were looked at, and takes 46.5; radius_kernel 44.2.  Only rows
        // that hide their mass from the tokens looked at still cost that.  Rows with radii of 0.018 throughout: radius_kernel 43.3, by
        // the radii alone, above 1/8, 45.6, so 41.0.  Active caps on every row, radii of 0.0025: 42.9 and 46.3, bf16 39.7 and 43.2.)
        // A wave without weight in the row (its tokens masked, say) takes the widths' sums and marks nothing.
        // Token widths of a row whose largest probability is at most 1/8 need 1/S as one float (1 - x to 1e-8).
        const bool split = (double)Elt<T>::exp2_ref(mc, n == -INFINITY ? 0.f : n) > 0.125 * S;
        auto am1_of = [&](float v) {
            if constexpr (SCALED) return am1_scaled(v, am1_max);
            else return radius_am1<T, UNIT>(v, kappa, rmax, am1_max);
        };
        // (an infinite radius may not go through the matrix cores; looked for ahead of the pass, all vectors at once)
        bool widen = MATRIX && quads;                              // uniform over the wave
        if (MATRIX && quads) {
            uint32_t huge = 0u;
#pragma unroll
            for (int j = 0; j < NVEC; ++j) {
                if (j < nch) {
                    u32x4 r = sm_next[j * THREADS + tid];
                    if ((j + 1) * CHUNK > V) E::zero_tail(r, (j * THREADS + tid) * EPV, V);   // uniform
                    huge = pk_max3(j == 0 ? pk_max3(r.x, r.x, r.y) : pk_max3(huge, r.x, r.y), r.z, r.w);
                }
                if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            widen = __builtin_amdgcn_ballot_w64(any_huge(huge)) == 0;
        }
        bool lean = false, weightless = false;                     // uniform over the wave
        if (!top && (!MATRIX || widen)) {
            lean = !A.normalize;
            if (A.normalize) {
                // (the raw radius of the lane's first slot; bf16, transposed: token l & 3 of the quad's first lane)
                const float raw = sizeof(T) == 4 ? bits_f(sm_next[tid].x)
                                                 : bits_f((uint32_t)reinterpret_cast<const uint16_t*>(sm_next)[(tid & ~3) * EPV + (tid & 3)] << 16);
                const float am1 = am1_of(SCALED ? raw * kBf16Scale : raw), Suf = uniform_f((float)Su), Vf = (float)V;
                weightless = etop * Vf < 0x1p-30f * Suf;
                const float enough = kExpectInactive * 64.0f * Suf, share = e[0] * Vf * (am1 * __builtin_amdgcn_rcpf(1.0f + am1));
                lean = weightless || wave_sum_f(fminf(share, 0.25f * enough)) > enough;
            }
        }
        float sum_pl = 0.f;
        constexpr int GROUP = sizeof(T) == 2 ? 2 : 4;              // vectors taken at a time
        // the pass over the vectors, in an instance of its own per kind (0: all five sums, 1: the widths', 2: those with 1 - x from
        // the two-part 1 / S), each with row constants of its own: what the instances have in common is otherwise formed for all
        // tokens ahead of the branch, and spilled
        auto pass = [&](auto kind) {
            constexpr int KIND = decltype(kind)::value;
            FuseRow f = fr;
            if (KIND > 0) asm volatile("" : "+v"(f.nih), "+v"(f.nil));
#pragma unroll
            for (int g = 0; g < NVEC; g += GROUP) {
                u32x4 rb[GROUP];
#pragma unroll
                for (int u = 0; u < GROUP; ++u) rb[u] = sm_next[(g + u) * THREADS + tid];
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (has_next) {
#pragma unroll
                    for (int u = 0; u < GROUP; ++u) fetch(next, g + u, tid);
                }
#pragma unroll
                for (int u = 0; u < GROUP; ++u) {
                    const int j = g + u;
                    if (j < nch) {                                     // uniform: the vectors hold tokens
                        if ((j + 1) * CHUNK > V) E::zero_tail(rb[u], (j * THREADS + tid) * EPV, V);
                        float rv[EPV];                                 // SCALED: times kBf16Scale
                        if (MATRIX && (KIND > 0 || __builtin_expect(widen, true))) {
                            if constexpr (SCALED) bf16_scaled(rb[u], bf16_scale(tid), rv);
                            else if constexpr (MATRIX) bf16_widened(rb[u], bf16_unit(tid), rv);
                        } else {
                            E::unpack(rb[u], rv);
                            if (MATRIX && quads) {
#pragma unroll
                                for (int k = 0; k < EPV; k += 4) quad_transpose(rv[k], rv[(k + 1) % EPV], rv[(k + 2) % EPV], rv[(k + 3) % EPV], tid);
                            }
                            if constexpr (SCALED) {
#pragma unroll
                                for (int k = 0; k < EPV; ++k) rv[k] *= kBf16Scale;
                            }
                        }
                        if constexpr (KIND > 0) {
#pragma unroll
                            for (int k = 0; k < EPV; ++k) {
                                const float ek = e[j * EPV + k], am1 = am1_of(rv[k]);
                                float om = fmaf(ek, f.nih, 1.0f);
                                if constexpr (KIND == 2) om = fmaf(ek, f.nil, om);
                                const float du = fmaf(am1, -ek * f.nih, 1.0f), dl = fmaf(am1, om, 1.0f);
                                const float g1 = ek * __builtin_amdgcn_rcpf(du * dl);
                                sum_pl = fmaf(g1, du, sum_pl);
                                const double dw = (double)((am1 * (am1 + 2.0f)) * (g1 * om));
                                q[1] += dw;
                                q[3] = fma(dw, dw, q[3]);
                            }
                        } else {
#pragma unroll
                            for (int k = 0; k < EPV; ++k) {
                                float pl, w;                               // (a slot past the row's end holds e = 0: both are 0)
                                fuse_token_am1(e[j * EPV + k], am1_of(rv[k]), f, pl, w);
                                const double dl = (double)pl, dw = (double)w;
                                q[0] += dl; q[1] += dw;
                                q[2] = fma(dl, dl, q[2]); q[3] = fma(dw, dw, q[3]); q[4] = fma(dl, dw, q[4]);
                            }
                        if (__builtin_expect(search, false)) {
#pragma unroll
                            for (int k = 0; k < EPV; ++k) {
                                const bool is = e[j * EPV + k] == etop;
                                raw_top = is ? rv[k] : raw_top;
                                found = found || is;
                            }
                        }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        // (what the branches expect decides what lies next to each other: a call of a few rows waits for its instructions to
        // arrive, and longer for those behind a jump)
        if (__builtin_expect(lean, true)) {
            if (ARGMAX || __builtin_expect(split, false)) pass(std::integral_constant<int, 2>{});
            else pass(std::integral_constant<int, 1>{});
        } else {
            pass(std::integral_constant<int, 0>{});
        }
        if (found) pk[done].raw_top = SCALED ? raw_top / kBf16Scale : raw_top;   // (one lane of the workgroup; the quotient is exact)
        {
            const double f2 = fw * fw;                             // to row units
            if (lean) {
                put((double)sum_pl * fw, 0, lane); put(q[1] * fw, 1, lane); put(q[3] * f2, 3, lane);
                // (the fifth sum's slots hold anything; the constant through an empty asm, or it is held through the row loop)
                int nan_hi = 0x7ff80000;
                asm volatile("" : "+v"(nan_hi));
                if ((lane & 7) == 0) sm_red[wave][2 * 8 + (lane >> 3)] = weightless ? 0.0 : __hiloint2double(nan_hi, nan_hi);
                if (weightless) put(0.0, 4, lane);
            } else {
                put(q[0] * fw, 0, lane); put(q[1] * fw, 1, lane);
                put(q[2] * f2, 2, lane); put(q[3] * f2, 3, lane); put(q[4] * f2, 4, lane);
            }
        }
        if (!has_next) break;
        pos = npos; h = nh;
        if constexpr (THREADS < 1024) priority_by_progress(done + 1, count);
    }
    {
        const int lane = my_tid() & 63;
        const double v = get(lane);
        if ((lane & 7) == 0 && lane < 8 * NQ) sm_tot[(count - 1) & 1][wave][lane >> 3] = v;
    }
    __syncthreads();
    if (wave == 0) park(count - 1, (count - 1) & 1);
    __syncthreads();
    // ---- a lane per row ---------------------------------------------------------------------------------------------------
    auto stats_of = [&](int at, bool& known) {
        RowStats st;
        known = true;
        st.S = pk[at].S; st.Z = 0.0; st.n = pk[at].n; st.nt = 0.f; st.mc = pk[at].mc;
#pragma unroll
        for (int i = 0; i < 5; ++i) st.q[i] = pk[at].q[i];
        st.kl = 0.0; st.kw = 0.0; st.mode = kSumsFull;
        if (st.q[2] != st.q[2]) {                         // the widths' sums, and whether they do
            const double Sl = st.q[0] / st.S, Su = Sl + st.q[1] / st.S;
            known = !A.normalize || (Sl <= A.cap_lo * (1.0 - kCapGuard) && Su >= A.cap_hi * (1.0 + kCapGuard));
            st.mode = kSumsWidthOnly;
            st.q[0] = 0.0; st.q[2] = 0.0; st.q[4] = 0.0;
        }
        return st;
    };
    auto row_of = [&](int at) { return (int64_t)(at % H) * P + blockIdx.x + (int64_t)(at / H) * step; };
    auto finish = [&](int at, const RowStats& st, auto again) {
        return finish_radius_row<T, ARGMAX>(A, row_of(at), pk_id[ARGMAX ? at : 0], st, pk[at].raw_top, &pk_flag[at], again);
    };
    constexpr uint8_t kFull = 1, kExact = 2;                       // what a row is taken again with: all sums in fp32, in fp64
    auto crowded = [&](const RowStats& st) {
        return [&](const RowScore& rs) {
            const double etop = (double)Elt<T>::exp2_ref(st.mc, st.n == -INFINITY ? 0.f : st.n);
            const double Vd = (double)V, mean = rs.omega / Vd;
            return !(rs.sigma * rs.sigma >= kCrowded * mean * mean) || (A.precise_flat && etop * Vd <= 2.0 * st.S);
        };
    };
    // (no outputs: the statistics alone, for the Ensemble's second sweep, which looks after its own flat rows)
    const bool outputs = A.p_lo || A.p_mid || A.p_hi || A.omega || A.sigma || A.score || A.flags;
    {
        const int t = my_tid();
        if (t < count) {
            bool known;
            const RowStats st = stats_of(t, known);
            if (!known) {
                pk_fp64[t] = kFull;
            } else if (!outputs) {
                pk_fp64[t] = 0;
                A.stats[row_of(t)] = st;
            } else {
                pk_fp64[t] = finish(t, st, crowded(st)) ? kExact : 0;
            }
        }
    }
    __syncthreads();
    for (int at = 0; at < count; ++at) {
        if (!pk_fp64[at]) continue;                                // uniform
        bool known;
        RowStats st = stats_of(at, known);
        if (pk_fp64[at] == kFull) {
            radius_row_full<T, THREADS, UNIT>(A, row_of(at), sm_red, st);
            __syncthreads();
            if (my_tid() == 0) {
                pk_fp64[at] = outputs && finish(at, st, crowded(st)) ? kExact : 0;
                if (!outputs) A.stats[row_of(at)] = st;
            }
            __syncthreads();
            if (!pk_fp64[at]) continue;
        }
        radius_row_fp64<T, THREADS>(A, row_of(at), sm_red, st);
        if (my_tid() == 0) finish(at, st, NeverAgain{});
    }
    if (votes) vote_of_positions(pk_flag, H, (int)mine, step, votes);
}

template <typename T, int THREADS, int NVEC, bool UNIT, bool ARGMAX, bool WIDE, bool LEAN>
constexpr auto radius_entry()
{
    if constexpr (LEAN) return &radius_lean_kernel<T, THREADS, NVEC, UNIT, ARGMAX>;
    else return &radius_kernel<T, THREADS, NVEC, UNIT, ARGMAX, WIDE>;
}

template <typename T, int THREADS, int NVEC, bool UNIT, bool ARGMAX, bool WIDE, bool LEAN>
hipError_t launch_radius_cfg(const RowArgs& a, int heads, uint8_t* votes, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    constexpr int kPerUnit = 1024 / THREADS;                       // workgroups a compute unit holds
    const int64_t resident = (int64_t)kPerUnit * compute_units(), positions = a.N / heads;
    constexpr auto kernel = radius_entry<T, THREADS, NVEC, UNIT, ARGMAX, WIDE, LEAN>();
    // Several heads: the rows of a position in one workgroup, which takes the vote, or -- where the chip then goes through
    // fewer rows in turn -- every row for itself and the vote in a launch of its own.  (fp32, by position / by row: 8 positions
    // of 8 heads 1024 tokens 31.8 / 10.8 us, 16384 tokens 49.2 / 13.5, 32768 tokens 79.8 / 19.4; 300 of 5 heads 1024 tokens
    // 23.6 / 14.9, 16384 tokens 54.3 / 43.4; 600 of 3 heads 32768 tokens 102 / 97.)  Small workgroups slow each other down when
    // all places are taken: half the rows in turn are wanted (2048 of 3 heads, 1024 tokens, two thirds: 22.1 / 23.9); of the large
    // ones a tenth less is enough (2100 of 2 heads, 32768 tokens bf16, 17 instead of 18: 162 / 167).
    const int64_t turns = (positions + resident - 1) / resident * heads, turns_by_row = (a.N + resident - 1) / resident;
    const bool by_row = heads > 1 && (THREADS < 512 ? 2 * turns_by_row <= turns : 10 * turns_by_row <= 9 * turns);
    if (by_row && !votes) heads = 1;
    if (by_row && votes) {
        const hipError_t e = launch_radius_cfg<T, THREADS, NVEC, UNIT, ARGMAX, WIDE, LEAN>(a, 1, nullptr, stream, ev_start, ev_stop);
        return e != hipSuccess ? e : launch_vote(a.flags, heads, positions, votes, stream);
    }
    constexpr unsigned lds = NVEC * 16u * THREADS;                 // 4 to 128 KiB
    if (lds > 32u * 1024u) {
        // with the static arrays above the default limit: raised once per device and instance
        static std::mutex guard;
        static bool raised[64] = {};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        std::lock_guard<std::mutex> lock(guard);
        if (!raised[dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            raised[dev] = true;
        }
    }
    const int64_t per_wg = radius_rows<THREADS>() / heads;         // positions (>= 2: heads <= 8)
    const int64_t g = whole_rounds(a.N / heads, per_wg, resident);
    const dim3 grid((unsigned)g), block(THREADS);
    if (ev_start && ev_stop)
        hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, ev_start, ev_stop, 0, a, heads,
                              votes);
    else
        hipLaunchKernelGGL(kernel, grid, block, lds, stream, a, heads, votes);
    return hipGetLastError();
}
template <typename T, int THREADS, int NVEC, bool WIDE>
hipError_t launch_radius_tile(const RowArgs& a, int heads, uint8_t* votes, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    const bool argmax = a.ids == nullptr && (a.p_lo || a.p_mid || a.p_hi);
    // radius_lean_kernel where rows follow one another: a call that has a place for every row waits for one row's instructions to
    // arrive, of which there are more then.  How many rows it takes to pay, by the lanes of a row (us, radius_kernel / radius_lean_kernel):
    // fp32, 64 lanes not at all (2048 tokens, 4500 rows 24.2 / 24.3; 1024 tokens, 9600 rows 25.7 / 26.1), from 128 lanes on more than
    // places (8000 tokens, 800 rows 20.2 / 19.8, 1600 rows 26.7 / 26.2; 16384 tokens, 400 rows 18.5 / 18.7, 520 rows 22.6 / 22.0);
    // bf16, 64 lanes full tiles and one and a half rows to a place (4096 tokens, 4500 rows 33.6 / 34.0, 6600 rows 41.8 / 40.8; 2500 tokens, 16384 rows
    // 61.7 / 62.1), 128 lanes more than places (8000 tokens, 1600 rows 26.4 / 26.5, 2200 rows 32.2 / 31.6), 256 lanes more than half
    // (16384 tokens, 400 rows 16.9 / 17.4, 520 rows 21.1 / 19.9), without drafted ids, and from 512 on, more than compute units (16384 tokens, 300
    // rows without ids 17.9 / 17.2; 32768 tokens, 270 rows 25.8 / 24.0).
    // Not with fp32 rows without drafted ids, which spill with it (2048 x 4096 22.8 and 25.3), nor with a clamp so small that no wave would
    // expect inactive caps (2048 x 16384 bf16 44.3 and 46.6).
    if constexpr (!WIDE) {
        constexpr bool B16 = sizeof(T) == 2;
        const int64_t units = compute_units(), places = (1024 / THREADS) * units;
        const bool follow = THREADS == 64  ? B16 && 2 * a.N > 3 * places && 4 * (int64_t)a.V > 3 * (int64_t)(NVEC * THREADS * Elt<T>::kPerVec)
                          : !B16 || THREADS == 128 ? a.N > places
                          : THREADS == 256 && !argmax ? 2 * a.N > places
                                           : a.N > units;
        if (follow && !(argmax && sizeof(T) == 4) && (a.am1_max > kExpectInactive || !a.normalize)) {
            if constexpr (sizeof(T) == 2) {
                if (argmax) return a.kappa == 1.0 ? launch_radius_cfg<T, THREADS, NVEC, true, true, false, true>(a, heads, votes, stream, ev_start, ev_stop)
                                                  : launch_radius_cfg<T, THREADS, NVEC, false, true, false, true>(a, heads, votes, stream, ev_start, ev_stop);
            }
            return a.kappa == 1.0 ? launch_radius_cfg<T, THREADS, NVEC, true, false, false, true>(a, heads, votes, stream, ev_start, ev_stop)
                                  : launch_radius_cfg<T, THREADS, NVEC, false, false, false, true>(a, heads, votes, stream, ev_start, ev_stop);
        }
    }
    if (a.kappa == 1.0) return argmax ? launch_radius_cfg<T, THREADS, NVEC, true, true, WIDE, false>(a, heads, votes, stream, ev_start, ev_stop)
                                      : launch_radius_cfg<T, THREADS, NVEC, true, false, WIDE, false>(a, heads, votes, stream, ev_start, ev_stop);
    return argmax ? launch_radius_cfg<T, THREADS, NVEC, false, true, WIDE, false>(a, heads, votes, stream, ev_start, ev_stop)
                  : launch_radius_cfg<T, THREADS, NVEC, false, false, WIDE, false>(a, heads, votes, stream, ev_start, ev_stop);
}
template <typename T, int NVEC, bool WIDE>
hipError_t launch_radius_lanes(const RowArgs& a, int heads, uint8_t* votes, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    // As many lanes as the row takes at NVEC vectors each -- or, where there is a row per compute unit at most (two, if that
    // leaves a lane two vectors), at one vector each, up to 256 lanes: then a call waits for one row's chain of instructions, and
    // fewer tokens per lane make it shorter.  (Without / with, 8 rows of 4096 tokens bf16 12.1 / 9.3 us, fp32 10.0 / 9.1; 300
    // rows 12.9 / 11.9 and 12.0 / 11.1, of 1024 tokens fp32 9.8 / 9.8, bf16 10.0 / 10.4; 1000 rows of 4096 bf16 13.5 / 16.6.  512
    // lanes, 8 rows of 4096 bf16: 10.2.)
    const int vecs = (a.V + Elt<T>::kPerVec - 1) / Elt<T>::kPerVec;
    const int vecs_per_lane = a.N <= (vecs >= 512 ? 2 : 1) * compute_units() ? 1 : NVEC;
    if (vecs <= 64 * vecs_per_lane) return launch_radius_tile<T, 64, NVEC, WIDE>(a, heads, votes, stream, ev_start, ev_stop);
    if (vecs <= 128 * vecs_per_lane) return launch_radius_tile<T, 128, NVEC, WIDE>(a, heads, votes, stream, ev_start, ev_stop);
    if (vecs <= 256 * NVEC) return launch_radius_tile<T, 256, NVEC, WIDE>(a, heads, votes, stream, ev_start, ev_stop);
    if (vecs <= 512 * NVEC) return launch_radius_tile<T, 512, NVEC, WIDE>(a, heads, votes, stream, ev_start, ev_stop);
    if (vecs <= 1024 * NVEC) return launch_radius_tile<T, 1024, NVEC, WIDE>(a, heads, votes, stream, ev_start, ev_stop);
    return hipErrorInvalidValue;
}
template <typename T>
hipError_t launch_radius_typed(const RowArgs& a, int heads, uint8_t* votes, hipStream_t stream, hipEvent_t ev_start,
                               hipEvent_t ev_stop)
{
    if (!wide_radius(a)) return launch_radius_lanes<T, kRadVecs, false>(a, heads, votes, stream, ev_start, ev_stop);
    if constexpr (sizeof(T) == 2) {
        if (a.V <= 1024 * kRadVecsWide16 * Elt<T>::kPerVec)
            return launch_radius_lanes<T, kRadVecsWide16, true>(a, heads, votes, stream, ev_start, ev_stop);
        if (a.V > max_vocab(1)) return hipErrorInvalidValue;
        return launch_radius_tile<T, 1024, kRadVecs, true>(a, heads, votes, stream, ev_start, ev_stop);
    } else {
        return launch_radius_lanes<T, kRadVecs, true>(a, heads, votes, stream, ev_start, ev_stop);
    }
}

}  // namespace

bool radius_quantify_fits(const RowArgs& args) { return args.radius != nullptr && args.V > kTinyVocab; }

hipError_t launch_radius_quantify(int dtype, const RowArgs& args, int heads, uint8_t* votes, hipStream_t stream,
                                  hipEvent_t ev_start, hipEvent_t ev_stop)
{
    if (args.N <= 0) return hipSuccess;
    if (!radius_quantify_fits(args) || heads < 1 || (votes && !args.flags)) return hipErrorInvalidValue;
    return dtype == 0 ? launch_radius_typed<float>(args, heads, votes, stream, ev_start, ev_stop)
                      : launch_radius_typed<bf16_t>(args, heads, votes, stream, ev_start, ev_stop);
}

}  // namespace ciar
