// Device-side helpers shared by the gfx950 kernels of the library: element types, exact-by-construction
// exponentials, wave reductions, the per-token InterFuse arithmetic and the per-row finishing formulas.
// Internal; included by the .hip files only.
#pragma once

#include "ciar_internal.h"

#include <limits.h>
#include <atomic>
#include <math.h>
#include <type_traits>

namespace ciar {
namespace {


// log2(e) split so that the low part is positive: x * hi + x * lo stays -inf for x = -inf.
constexpr float  kLog2eHi = 1.44269490242004394531f;   // largest float below log2(e)
constexpr float  kLog2eLo = 1.384689195e-7f;           // log2(e) - kLog2eHi
constexpr double kLn2 = 0.69314718055994530942;

__device__ __forceinline__ float bits_f(uint32_t u) { return __uint_as_float(u); }

// A value that is the same in every lane of the wave, moved to a scalar register.
__device__ __forceinline__ float uniform_f(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

constexpr int kNonTemporal = 2;        // cache policy of global_load_lds for rows that are used once

// 16 bytes as loaded: a native vector type, so it can be read through an address-space pointer.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
using gbytes = const __attribute__((address_space(1))) char*;
using gvec = const __attribute__((address_space(1))) u32x4*;

// 2^(x log2(e) - n) for an integer-valued reference n.  x * hi - n is exact inside the FMA and is
// rounded at the magnitude of the (small) result; the low part of log2(e) is added by a second FMA.
__device__ __forceinline__ float exp2_ref(float x, float n)
{
    return __builtin_amdgcn_exp2f(fmaf(x, kLog2eLo, fmaf(x, kLog2eHi, -n)));
}

// Integer reference for a set of logits whose maximum is m: the next integer above m * log2(e), so
// every 2^(x log2e - n) is <= 1 (up to rounding).  -inf (nothing but masked tokens) maps to -inf.
// Logits of large magnitude: from 2^24 on n is a multiple of 2, 4, ..., 128 (up to 2^31), so that the largest token's exponential is
// anything from 2^-92 to 2^92 instead of 1/2 to 1.  Sums, reciprocals and token widths hold that, and a row masked throughout with
// -1e9, or a token forced with 1e9, comes out right (any logit up to a magnitude of 1.48e9; beyond, those whose exponential the
// rounding of n leaves in range).  Powers of 1 / S do not hold it, and ask ref_is_near.  Further up that exponential can overflow,
// and a wave of masked tokens (-1e10, say) would outweigh the others': where m log2(e) lies that far above the rounded n, n is
// raised by more than its own rounding (by a finite number: n may be -inf, and stays that).
__device__ __forceinline__ float ref_of(float m)
{
    const float n = ceilf(m * 1.44269504f);
    return fmaf(m, 1.44269504f, -n) > 100.f ? fmaf(fminf(fabsf(n), 0x1p127f), 0x1p-22f, n) : n;
}
__device__ __forceinline__ bool ref_is_near(float n) { return !(fabsf(n) >= 0x1p24f); }

// Maximum of three logits.  (None is a signalling NaN: plain v_max3_f32, without the quieting of each operand that fmaxf
// adds for values the compiler knows nothing about.)
__device__ __forceinline__ float max3(float a, float b, float c)
{
    float m;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(c));
    return m;
}
__device__ __forceinline__ float max2(float a, float b)
{
    float m;
    asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
    return m;
}
template <int N>
__device__ __forceinline__ float max_of(const float (&v)[N])
{
    static_assert(N >= 4 && N % 2 == 0, "pairs");
    float m = max3(v[0], v[0], v[1]);
#pragma unroll
    for (int i = 2; i < N; i += 2) m = max3(m, v[i], v[i + 1]);
    return m;
}

// 1 / x for an ordinary positive x, to the last bit or so (hardware estimate and two Newton steps: a third of the
// instructions of the division, which also covers operands at the ends of the range)
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// Most binary orders that a wave's units lie below its row's when the row's sum is taken to them: with logits of 1e9 the sum itself
// is up to 2^100 (2^1000 S overflowed, and recip of that is no number); the wave's tokens weigh nothing from 2^200 on.
constexpr float kFarUnits = 900.f;
// 2^k as a double for an integer-valued float difference k <= 0 (clamped: below 2^-1000 it is 0 anyway)
__device__ __forceinline__ double pow2_of(float k) { return ldexp(1.0, (int)fmaxf(k, -1000.f)); }

// bf16 logits x: kBf16Scale (15 significant bits) times x is exact in fp32, and kBf16Scale * kBf16ToLog2e is log2(e) to 1.2e-13
// relative, so 2^(x log2(e) - n) takes one FMA whose only error is its own rounding.  (fp32 logits: exp2_ref.)
constexpr float kBf16Scale = 1.52874755859375f;        // = kBf16ScaleHi + kBf16ScaleLo, each a bf16 number
constexpr float kBf16ToLog2e = 0.94371045f;
constexpr uint32_t kBf16ScaleHi = 0x3fc4u, kBf16ScaleLo = 0xbb24u;
__device__ __forceinline__ float exp2_scaled(float z, float n)         // z = kBf16Scale x
{
    return __builtin_amdgcn_exp2f(fmaf(z, kBf16ToLog2e, -n));
}

template <typename T> struct Elt;
template <> struct Elt<float> {
    static constexpr int kPerVec = 4;
    static constexpr double kLog2e = (double)kLog2eHi + (double)kLog2eLo;          // as the exponentials have it
    __device__ static __forceinline__ float exp2_ref(float x, float n) { return ciar::exp2_ref(x, n); }
    static constexpr uint32_t kNegInfWord = 0xff800000u;
    __device__ static __forceinline__ void unpack(const u32x4& r, float* o)
    {
        o[0] = bits_f(r.x); o[1] = bits_f(r.y); o[2] = bits_f(r.z); o[3] = bits_f(r.w);
    }
    // Replace elements with index >= V of a vector that starts at element `base` by -inf.
    __device__ static __forceinline__ void mask_tail(u32x4& r, int base, int V)
    {
        if (base + 0 >= V) r.x = kNegInfWord;
        if (base + 1 >= V) r.y = kNegInfWord;
        if (base + 2 >= V) r.z = kNegInfWord;
        if (base + 3 >= V) r.w = kNegInfWord;
    }
    // ... by zero.
    __device__ static __forceinline__ void zero_tail(u32x4& r, int base, int V)
    {
        if (base + 0 >= V) r.x = 0u;
        if (base + 1 >= V) r.y = 0u;
        if (base + 2 >= V) r.z = 0u;
        if (base + 3 >= V) r.w = 0u;
    }
};
struct bf16_t { uint16_t bits; };
template <> struct Elt<bf16_t> {
    static constexpr int kPerVec = 8;
    static constexpr double kLog2e = (double)kBf16Scale * (double)kBf16ToLog2e;    // as the exponentials have it
    // (the same number, bit for bit, as from the matrix cores' product: see bf16_scaled)
    __device__ static __forceinline__ float exp2_ref(float x, float n) { return exp2_scaled(x * kBf16Scale, n); }
    static constexpr uint32_t kNegInfWord = 0xff80ff80u;
    __device__ static __forceinline__ void unpack(const u32x4& r, float* o)
    {
        o[0] = bits_f(r.x << 16); o[1] = bits_f(r.x & 0xffff0000u);
        o[2] = bits_f(r.y << 16); o[3] = bits_f(r.y & 0xffff0000u);
        o[4] = bits_f(r.z << 16); o[5] = bits_f(r.z & 0xffff0000u);
        o[6] = bits_f(r.w << 16); o[7] = bits_f(r.w & 0xffff0000u);
    }
    // (by -inf, or by the pattern whose word is `fill`)
    __device__ static __forceinline__ uint32_t mask_word(uint32_t w, int base, int V, uint32_t fill)
    {
        if (base >= V) return fill;
        if (base + 1 >= V) return (w & 0x0000ffffu) | (fill & 0xffff0000u);
        return w;
    }
    __device__ static __forceinline__ void mask_tail(u32x4& r, int base, int V, uint32_t fill = kNegInfWord)
    {
        r.x = mask_word(r.x, base + 0, V, fill); r.y = mask_word(r.y, base + 2, V, fill);
        r.z = mask_word(r.z, base + 4, V, fill); r.w = mask_word(r.w, base + 6, V, fill);
    }
    __device__ static __forceinline__ uint32_t zero_word(uint32_t w, int base, int V)
    {
        return w & ((base < V ? 0x0000ffffu : 0u) | (base + 1 < V ? 0xffff0000u : 0u));
    }
    __device__ static __forceinline__ void zero_tail(u32x4& r, int base, int V)
    {
        r.x = zero_word(r.x, base + 0, V); r.y = zero_word(r.y, base + 2, V);
        r.z = zero_word(r.z, base + 4, V); r.w = zero_word(r.w, base + 6, V);
    }
};

// bf16 rows widened by the matrix cores.  What a token of a bf16 row costs on the vector ALUs beyond its exponential and its
// sums is unpacking it from its half of a word and taking it to base 2 (two multiply-adds): three issues of eight.  A 4 x 4
// matrix product per four lanes, (the lanes' four tokens each) x (kBf16Scale on the diagonal), does the unpacking and the exact
// scaling of four tokens per lane in one issue per bf16 part of kBf16Scale, next to the vector ALUs' work: with the FMA
// that is left, one and a half issues per token for three.  The products are exact, so the result is the number that
// x * kBf16Scale gives, bit for bit.
// Slots: the tokens of a quad's four lanes come back transposed: slot 4 g + r of lane l holds token 4 g + (l & 3) of lane
// (l & ~3) + r's vector.  Sums over a row do not care; whoever wants a slot's token index asks slot_base and slot_step.
// An infinity would make its three neighbours 0 * inf: rows that may hold one are widened on the vector ALUs (wave_top; sums
// that come out as no number).
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
struct Bf16Scale { s16x4 hi, lo; };                                // this lane's column of the two diagonal matrices
__device__ __forceinline__ Bf16Scale bf16_scale(int lane)
{
    const uint32_t up = (uint32_t)(lane & 1) * 16u;
    const bool first = (lane & 2) == 0;
    const uint32_t h = kBf16ScaleHi << up, l = kBf16ScaleLo << up;
    return {__builtin_bit_cast(s16x4, u32x2{first ? h : 0u, first ? 0u : h}),
            __builtin_bit_cast(s16x4, u32x2{first ? l : 0u, first ? 0u : l})};
}
__device__ __forceinline__ void bf16_scaled(const u32x4& r, const Bf16Scale& m, float* z)
{
    const s16x4 a = __builtin_bit_cast(s16x4, u32x2{r.x, r.y}), b = __builtin_bit_cast(s16x4, u32x2{r.z, r.w});
    f32x4 za = {0.f, 0.f, 0.f, 0.f}, zb = za;
    za = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, m.hi, za, 0, 0, 0);
    zb = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(b, m.hi, zb, 0, 0, 0);
    za = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, m.lo, za, 0, 0, 0);
    zb = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(b, m.lo, zb, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) { z[k] = za[k]; z[4 + k] = zb[k]; }
}
// the tokens as they are, in the same slots (a diagonal of ones: one product)
__device__ __forceinline__ s16x4 bf16_unit(int lane)
{
    const uint32_t h = 0x3f80u << ((uint32_t)(lane & 1) * 16u);
    const bool first = (lane & 2) == 0;
    return __builtin_bit_cast(s16x4, u32x2{first ? h : 0u, first ? 0u : h});
}
__device__ __forceinline__ void bf16_widened(const u32x4& r, const s16x4& m, float* z)
{
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const f32x4 za = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, u32x2{r.x, r.y}), m, zero, 0, 0, 0);
    const f32x4 zb = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, u32x2{r.z, r.w}), m, zero, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) { z[k] = za[k]; z[4 + k] = zb[k]; }
}
// Token index of slot k (of 4 g + r) of this thread's vector, from the first token of the workgroup's vectors: slot_base + 4 g +
// slot_step r; `quads` = the slots are transposed.
__device__ __forceinline__ int slot_base(bool quads, int tid, int per_vec)
{
    return quads ? (tid & ~3) * per_vec + (tid & 3) : tid * per_vec;
}
__device__ __forceinline__ int slot_step(bool quads, int per_vec) { return quads ? per_vec : 1; }

// v[i] of lane j of a quad <-> v[j] of lane i: slots to tokens in order and back (two exchanges with a neighbour lane)
__device__ __forceinline__ void quad_transpose(float& v0, float& v1, float& v2, float& v3, int lane)
{
    auto swap = [](float& a, float& b, bool upper, auto ctrl) {   // the pair's lower lane gives b for the upper lane's a
        const float give = upper ? a : b;
        const float got = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(give), decltype(ctrl)::value, 0xf, 0xf, true));
        if (upper) a = got; else b = got;
    };
    const bool odd = (lane & 1) != 0, high = (lane & 2) != 0;
    constexpr std::integral_constant<int, 0xB1> by1{};             // quad_perm 1,0,3,2
    constexpr std::integral_constant<int, 0x4E> by2{};             // quad_perm 2,3,0,1
    swap(v0, v1, odd, by1);
    swap(v2, v3, odd, by1);
    swap(v0, v2, high, by2);
    swap(v1, v3, high, by2);
}

// The largest logit of a wave's bf16 words without unpacking them: as fp16 numbers bf16 patterns have the same order, and gfx950
// takes the maximum of three packed pairs in one issue (a quarter of an issue per token; unpacked: a half, and the
// unpacking).  Patterns that are infinities or no numbers in fp16 -- bf16 magnitudes from 2^121 on, masked tokens at -inf or the
// type's lowest value among them -- come through as such (`ordinary` is false in wave_top): then the wave's tokens are unpacked.
constexpr uint32_t kNoTokenWord = 0xfbfffbffu;                     // below every ordinary logit: padding
__device__ __forceinline__ uint32_t pk_max3(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t m;
    asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(m) : "v"(a), "v"(b), "v"(c));
    return m;
}
__device__ __forceinline__ bool any_huge(uint32_t w) { return (w & 0x7c00u) == 0x7c00u || (w & 0x7c000000u) == 0x7c000000u; }
template <int N>
__device__ __forceinline__ uint32_t top_words(const u32x4 (&v)[N])
{
    uint32_t m = kNoTokenWord;
#pragma unroll
    for (int j = 0; j < N; ++j) m = pk_max3(pk_max3(m, v[j].x, v[j].y), v[j].z, v[j].w);
    return m;
}

// ln of 2^(x log2(e) - n) in fp64, to stand next to sums of such numbers: with the log2(e) they are taken with, whose error a logit
// of 1e8 multiplies to 1e-5.
template <typename T>
__device__ __forceinline__ double ln_exp2(float x, double n) { return fma((double)x, Elt<T>::kLog2e, -n) * kLn2; }

template <typename T>
__device__ __forceinline__ float load_logit(const T* row, int i)
{
    if constexpr (sizeof(T) == 4) return reinterpret_cast<const float*>(row)[i];
    else return bits_f((uint32_t)reinterpret_cast<const uint16_t*>(row)[i] << 16);
}

// Element offset of row r from the start of a logit tensor, and the index of its drafted token (see RowArgs:
// several heads in one launch).  Rows are counted in 32 bits (the entry points reject more).
__device__ __forceinline__ int64_t row_offset(const RowArgs& A, int64_t r)
{
    if (A.head_rows == 0) return r * A.stride;
    const uint32_t h = (uint32_t)r / (uint32_t)A.head_rows;
    return (int64_t)h * A.head_stride + (int64_t)((uint32_t)r - h * (uint32_t)A.head_rows) * A.stride;
}
__device__ __forceinline__ int64_t ids_index(const RowArgs& A, int64_t r)
{
    return A.ids_period ? (int64_t)((uint32_t)r % (uint32_t)A.ids_period) : r;
}

// ---- wave reductions (fixed order: deterministic) ----------------------------------------------
//
// DPP row shifts and row broadcasts: they run on the vector ALU at full rate, whereas a shuffle
// (ds_bpermute) goes through the LDS crossbar and costs ~5x more per step.
// Pattern (wave64 = 4 rows of 16 lanes): row_shr 1, 2, 4, 8 leave each row's inclusive prefix in its
// lanes; row_bcast:15 adds a row's total into the next row (rows 1 and 3), row_bcast:31 adds lane 31
// into rows 2 and 3; every lane then holds its inclusive prefix over the wave and lane 63 the total,
// which readlane hands to every lane.

constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;

// value of the lane selected by CTRL, or `fill` where the selection is out of range / masked off
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_or(int fill, int v)
{
    return __builtin_amdgcn_update_dpp(fill, v, CTRL, ROW_MASK, 0xf, false);
}

// the same with 0 for lanes without a source, all rows written (no register has to be cleared for the result first)
template <int CTRL>
__device__ __forceinline__ int dpp_zero(int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
constexpr bool dpp_in_row(int ctrl) { return ctrl != 0x142 && ctrl != 0x143; }   // (not a broadcast from row to row)

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double v)
{
    if constexpr (ROW_MASK == 0xf && dpp_in_row(CTRL))
        return v + __hiloint2double(dpp_zero<CTRL>(__double2hiint(v)), dpp_zero<CTRL>(__double2loint(v)));
    const int lo = dpp_or<CTRL, ROW_MASK>(0, __double2loint(v));
    const int hi = dpp_or<CTRL, ROW_MASK>(0, __double2hiint(v));
    return v + __hiloint2double(hi, lo);           // lanes without a source add +0.0
}

// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ double wave_scan(double v)
{
    v = dpp_add<kRowShr1, 0xf>(v);
    v = dpp_add<kRowShr2, 0xf>(v);
    v = dpp_add<kRowShr4, 0xf>(v);
    v = dpp_add<kRowShr8, 0xf>(v);
    v = dpp_add<kRowBcast15, 0xa>(v);
    v = dpp_add<kRowBcast31, 0xc>(v);
    return v;
}

__device__ __forceinline__ double wave_sum(double v)
{
    v = wave_scan(v);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

// Three sums over the wave at once, handed to every lane, in two steps so that the values need not be there at the same
// time.  wave_sum3_put: two DPP steps leave every quad's sum in its lanes and the quad leaders put it into row `which`
// of the wave's 48 slots of LDS.  wave_sum3_get: lane l < 48 takes slot l and one reduction over each row of 16 lanes
// finishes all three (a wave's LDS operations complete in order: no barrier).  ~45 instructions where three
// reductions of one double each are ~110, and nothing is held in registers between the two steps.
__device__ __forceinline__ void wave_sum3_put(double v, double* slots, int which, int lane)
{
    v = dpp_add<0xB1, 0xf>(v);                     // lane ^ 1  (quad_perm 1,0,3,2)
    v = dpp_add<0x4E, 0xf>(v);                     // lane ^ 2  (quad_perm 2,3,0,1)
    if ((lane & 3) == 0) slots[16 * which + (lane >> 2)] = v;
}
__device__ __forceinline__ void wave_sum3_get(const double* slots, int lane, double& a, double& b, double& c)
{
    double x = slots[lane < 48 ? lane : 0];
    x = lane < 48 ? x : 0.0;
    x = dpp_add<kRowShr1, 0xf>(x);
    x = dpp_add<kRowShr2, 0xf>(x);
    x = dpp_add<kRowShr4, 0xf>(x);
    x = dpp_add<kRowShr8, 0xf>(x);
    const int lo = __double2loint(x), hi = __double2hiint(x);
    a = __hiloint2double(__builtin_amdgcn_readlane(hi, 15), __builtin_amdgcn_readlane(lo, 15));
    b = __hiloint2double(__builtin_amdgcn_readlane(hi, 31), __builtin_amdgcn_readlane(lo, 31));
    c = __hiloint2double(__builtin_amdgcn_readlane(hi, 47), __builtin_amdgcn_readlane(lo, 47));
}

// sum over lanes 0..15 (the first DPP row), handed to every lane of the wave
__device__ __forceinline__ double row16_sum(double v)
{
    v = dpp_add<kRowShr1, 0xf>(v);
    v = dpp_add<kRowShr2, 0xf>(v);
    v = dpp_add<kRowShr4, 0xf>(v);
    v = dpp_add<kRowShr8, 0xf>(v);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 15);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 15);
    return __hiloint2double(hi, lo);
}

// the same for a float
__device__ __forceinline__ float row16_sum_f(float v)
{
    v += __int_as_float(dpp_or<kRowShr1, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowShr2, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowShr4, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowShr8, 0xf>(0, __float_as_int(v)));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 15));
}

// the sum of a float over the wave, handed to every lane
__device__ __forceinline__ float wave_sum_f(float v)
{
    v += __int_as_float(dpp_or<kRowShr1, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowShr2, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowShr4, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowShr8, 0xf>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowBcast15, 0xa>(0, __float_as_int(v)));
    v += __int_as_float(dpp_or<kRowBcast31, 0xc>(0, __float_as_int(v)));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max(float v)
{
    // lanes without a source get their own value back: max(v, v) = v
    return max2(v, __int_as_float(dpp_or<CTRL, ROW_MASK>(__float_as_int(v), __float_as_int(v))));
}

__device__ __forceinline__ float wave_max(float v)
{
    v = dpp_max<kRowShr1, 0xf>(v);
    v = dpp_max<kRowShr2, 0xf>(v);
    v = dpp_max<kRowShr4, 0xf>(v);
    v = dpp_max<kRowShr8, 0xf>(v);
    v = dpp_max<kRowBcast15, 0xa>(v);
    v = dpp_max<kRowBcast31, 0xc>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// the same for top_words: the larger of the wave's two halves as a float; `ordinary` as above
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_pk_max(uint32_t v)
{
    const uint32_t o = (uint32_t)dpp_or<CTRL, ROW_MASK>((int)v, (int)v);
    return pk_max3(v, o, o);
}
__device__ __forceinline__ float wave_top(uint32_t v, bool& ordinary)
{
    v = dpp_pk_max<kRowShr1, 0xf>(v);
    v = dpp_pk_max<kRowShr2, 0xf>(v);
    v = dpp_pk_max<kRowShr4, 0xf>(v);
    v = dpp_pk_max<kRowShr8, 0xf>(v);
    v = dpp_pk_max<kRowBcast15, 0xa>(v);
    v = dpp_pk_max<kRowBcast31, 0xc>(v);
    const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    const float m = fmaxf(bits_f(u & 0xffff0000u), bits_f(u << 16));
    ordinary = !any_huge(u) && m > bits_f(kNoTokenWord & 0xffff0000u);
    return m;
}

// maximum over lanes 0..15 (the first DPP row), handed to every lane of the wave
__device__ __forceinline__ float row16_max(float v)
{
    v = dpp_max<kRowShr1, 0xf>(v);
    v = dpp_max<kRowShr2, 0xf>(v);
    v = dpp_max<kRowShr4, 0xf>(v);
    v = dpp_max<kRowShr8, 0xf>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 15));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_max(double v)
{
    // lanes without a source get their own value back
    const int lo = dpp_or<CTRL, ROW_MASK>(__double2loint(v), __double2loint(v));
    const int hi = dpp_or<CTRL, ROW_MASK>(__double2hiint(v), __double2hiint(v));
    return fmax(v, __hiloint2double(hi, lo));
}

__device__ __forceinline__ double wave_max(double v)
{
    v = dpp_max<kRowShr1, 0xf>(v);
    v = dpp_max<kRowShr2, 0xf>(v);
    v = dpp_max<kRowShr4, 0xf>(v);
    v = dpp_max<kRowShr8, 0xf>(v);
    v = dpp_max<kRowBcast15, 0xa>(v);
    v = dpp_max<kRowBcast31, 0xc>(v);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ int wave_min_i(int v)
{
    v = min(v, dpp_or<kRowShr1, 0xf>(v, v));
    v = min(v, dpp_or<kRowShr2, 0xf>(v, v));
    v = min(v, dpp_or<kRowShr4, 0xf>(v, v));
    v = min(v, dpp_or<kRowShr8, 0xf>(v, v));
    v = min(v, dpp_or<kRowBcast15, 0xa>(v, v));
    v = min(v, dpp_or<kRowBcast31, 0xc>(v, v));
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ int wave_max_i(int v)
{
    v = max(v, dpp_or<kRowShr1, 0xf>(v, v));
    v = max(v, dpp_or<kRowShr2, 0xf>(v, v));
    v = max(v, dpp_or<kRowShr4, 0xf>(v, v));
    v = max(v, dpp_or<kRowShr8, 0xf>(v, v));
    v = max(v, dpp_or<kRowBcast15, 0xa>(v, v));
    v = max(v, dpp_or<kRowBcast31, 0xc>(v, v));
    return __builtin_amdgcn_readlane(v, 63);
}

// Workgroup barrier for data exchanged through LDS only: waits for this wave's LDS operations and joins the barrier.
// __syncthreads() also waits for every outstanding load into LDS (its fence covers them), and with it for the rows that
// a kernel has in flight there while it works on the current one.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- per-token InterFuse arithmetic, shared by the streaming kernel and the dense export ------------

// Constants of one row for a scalar radius.  Units: e_i as held by the lane, S = sum e_i in the same units.
struct FuseRow {
    float cu;            // (a-1)/S:  du = 1 + (a-1) x = 1 + cu e
    float nih, nil;      // -1/S split in two floats:  1 - x = 1 + nih e + nil e  (exact to ~1e-15)
    float b, omb;        // b and 1-b:  dl = 1 - (1-b) x = b + (1-b)(1-x), free of cancellation as x -> 1
};

__device__ __forceinline__ FuseRow fuse_row_inv(double invS, double a, double b)
{
    FuseRow r;
    r.cu = (float)((a - 1.0) * invS);
    r.nih = (float)(-invS);
    r.nil = (float)(-invS - (double)r.nih);
    r.b = (float)b;
    r.omb = (float)(1.0 - b);
    return r;
}
__device__ __forceinline__ FuseRow fuse_row(double S, double a, double b) { return fuse_row_inv(1.0 / S, a, b); }

// One token of the scalar-radius interval pass:  g = e / (du dl), so that gl = g du and gw = g om (om = 1 - x)
// with p^l = (b/S) gl and w = p^u - p^l = ((a-b)/S) gw.
// SPLIT = form 1 - x with the two-float 1/S.  It matters only when some x is close to 1 (the relative
// error of 1 - x is 6e-8 x / (1 - x) without it); rows whose largest probability is at most 1/2 skip it.
template <bool SPLIT = true>
__device__ __forceinline__ void fuse_parts(float e, const FuseRow& r, float& g, float& du, float& om)
{
    om = SPLIT ? fmaf(e, r.nil, fmaf(e, r.nih, 1.0f)) : fmaf(e, r.nih, 1.0f);   // 1 - x
    du = fmaf(e, r.cu, 1.0f);
    const float dl = fmaf(om, r.omb, r.b);
    g = e * __builtin_amdgcn_rcpf(du * dl);
}

template <bool SPLIT = true>
__device__ __forceinline__ void fuse_token(float e, const FuseRow& r, float& gl, float& gw)
{
    float g, du, om;
    fuse_parts<SPLIT>(e, r, g, du, om);
    gl = g * du;
    gw = g * om;
}

// The complement of the width next to gl and gw:  ec = 1 - (p^u - p^l) = (1 - 2 (1-b) x (1-x)) / (du dl)
// (from a b = 1).  The numerator lies in [1/2, 1], so ec keeps its relative accuracy where the width itself
// rounds to 1: with a large radius every p^u_i is close to 1, the widths differ from each other by less
// than an fp32 ulp, and only the sums of ec resolve their standard deviation.
__device__ __forceinline__ void fuse_token_wide(float e, const FuseRow& r, float& gl, float& gw, float& ec)
{
    const float om = fmaf(e, r.nil, fmaf(e, r.nih, 1.0f));        // 1 - x
    const float x = -e * r.nih;
    const float du = fmaf(e, r.cu, 1.0f);
    const float dl = fmaf(om, r.omb, r.b);
    const float rc = __builtin_amdgcn_rcpf(du * dl);
    const float g = e * rc;
    gl = g * du;
    gw = g * om;
    ec = fmaf(-2.0f * r.omb, x * om, 1.0f) * rc;
}

// Tensor-radius mode (Sec. 3.2.3, the Interval Head: r = Softplus(raw)): r = min(kappa Softplus(raw), rmax) in
// fp32.  Softplus(raw) = max(raw, 0) + ln(1 + t), t = e^-|raw|.  With u = fl(1 + t) and d = u - 1 (exact),
// ln(1 + t) = ln(u) + ln(1 + (t - d) / u) = ln(u) + (t - d)(2 - u) to 3e-8 relative: |t - d| is at most half an
// ulp of u and 1/u = 2 - u + d^2/u, so the rounding of 1 + t is put back and small radii (raw << 0, where
// ln(u) alone would be a multiple of 1.2e-7) keep their relative accuracy.  t below half an ulp of 1: u = 1,
// ln(u) = 0 and the correction is t itself.
__device__ __forceinline__ float radius_r(float raw, float kappa, float rmax)
{
    const float t = __builtin_amdgcn_exp2f(-fabsf(raw) * 1.44269504f);
    const float u = 1.0f + t;
    const float d = u - 1.0f;
    const float lg = fmaf(__builtin_amdgcn_logf(u), 0.693147181f, (t - d) * (2.0f - u));
    return fminf(kappa * (fmaxf(raw, 0.f) + lg), rmax);
}

// The same radius in fp64 (one token per row: the reported token's interval).
__device__ __forceinline__ double radius_of(double raw, double kappa, double rmax)
{
    const double sp = raw > 0.0 ? raw + log1p(exp(-raw)) : log1p(exp(raw));
    return fmin(kappa * sp, rmax);
}

// a - 1 = e^r - 1 of a tensor-radius token, r = min(kappa Softplus(raw), rmax); am1_max = e^rmax - 1.
// UNIT (kappa = 1, the Interval Head as the paper defines it): e^Softplus(raw) = 1 + e^raw, so a - 1 = e^raw, capped:
// one exponential, no logarithm, and no cancellation in a - 1 however small the radius is.  (bf16: the same floats from the
// matrix cores' products, am1_scaled.)
__device__ __forceinline__ float am1_scaled(float z, float am1_max)     // z = kBf16Scale raw
{
    return fminf(__builtin_amdgcn_exp2f(z * kBf16ToLog2e), am1_max);
}
template <typename T, bool UNIT>
__device__ __forceinline__ float radius_am1(float raw, float kappa, float rmax, float am1_max)
{
    if constexpr (UNIT && sizeof(T) == 2) return am1_scaled(raw * kBf16Scale, am1_max);
    else if constexpr (UNIT) return fminf(__builtin_amdgcn_exp2f(fmaf(raw, kLog2eLo, raw * kLog2eHi)), am1_max);
    else return __builtin_amdgcn_exp2f(radius_r(raw, kappa, rmax) * 1.44269504f) - 1.0f;
}

// Tensor-radius token: pl = p^l_i S and w = (p^u_i - p^l_i) S in the units of e, from a - 1 alone.  With
// b = 1/a the lower bound's denominator times a is dl = 1 + (a-1)(1-x) (no cancellation: both terms >= 0), and
//   p^l S = e / dl,   p^u S = a e / du (du = 1 + (a-1) x),   (p^u - p^l) S = (a-1)(a+1) e (1-x) / (du dl),
// so that neither b nor a second reciprocal is needed.
__device__ __forceinline__ void fuse_token_am1(float e, float am1, const FuseRow& r, float& pl, float& w)
{
    const float om = fmaf(e, r.nil, fmaf(e, r.nih, 1.0f));        // 1 - x
    const float x = -e * r.nih;
    const float du = fmaf(am1, x, 1.0f);
    const float dl = fmaf(am1, om, 1.0f);
    const float g = e * __builtin_amdgcn_rcpf(du * dl);
    pl = g * du;
    w = (am1 * (am1 + 2.0f)) * (g * om);
}
template <typename T, bool UNIT>
__device__ __forceinline__ void fuse_token_rad(float e, float raw, const FuseRow& r, float kappa, float rmax,
                                               float am1_max, float& pl, float& w)
{
    fuse_token_am1(e, radius_am1<T, UNIT>(raw, kappa, rmax, am1_max), r, pl, w);
}

// The same with the complement of the width (see fuse_token_wide), in the same units:
// ec = 1 - (p^u_i - p^l_i) = (a - 2 (a-1) x (1-x)) / (du dl).
template <typename T, bool UNIT>
__device__ __forceinline__ void fuse_token_rad_wide(float e, float raw, const FuseRow& r, float kappa, float rmax,
                                                    float am1_max, float& pl, float& w, float& ec)
{
    const float am1 = radius_am1<T, UNIT>(raw, kappa, rmax, am1_max);
    const float om = fmaf(e, r.nil, fmaf(e, r.nih, 1.0f));        // 1 - x
    const float x = -e * r.nih;
    const float du = fmaf(am1, x, 1.0f);
    const float dl = fmaf(am1, om, 1.0f);
    const float rc = __builtin_amdgcn_rcpf(du * dl);
    const float g = e * rc;
    pl = g * du;
    w = (am1 * (am1 + 2.0f)) * (g * om);
    ec = fmaf(-2.0f * am1, x * om, am1 + 1.0f) * rc;
}

// The two with the choice made at run time (uniform over a launch).
struct RadiusMode { bool unit; float kappa, rmax, am1_max; };
__device__ __forceinline__ RadiusMode radius_mode(const RowArgs& A)
{
    return {A.kappa == 1.0, (float)A.kappa, (float)A.rmax, A.am1_max};
}
template <typename T>
__device__ __forceinline__ void fuse_token_rad(float e, float raw, const FuseRow& r, const RadiusMode& m, float& pl,
                                               float& w)
{
    if (m.unit) fuse_token_rad<T, true>(e, raw, r, m.kappa, m.rmax, m.am1_max, pl, w);
    else fuse_token_rad<T, false>(e, raw, r, m.kappa, m.rmax, m.am1_max, pl, w);
}
template <typename T>
__device__ __forceinline__ void fuse_token_rad_wide(float e, float raw, const FuseRow& r, const RadiusMode& m,
                                                    float& pl, float& w, float& ec)
{
    if (m.unit) fuse_token_rad_wide<T, true>(e, raw, r, m.kappa, m.rmax, m.am1_max, pl, w, ec);
    else fuse_token_rad_wide<T, false>(e, raw, r, m.kappa, m.rmax, m.am1_max, pl, w, ec);
}

// Vocabularies of at most this many tokens take fp64 token arithmetic (see fuse_sums_tiny, dro_row_tiny_kernel).
constexpr int kTinyVocab = 64;

// Per-row scalars of the quantifier from the five sums (fp64, one lane).
struct RowScore { double alpha_l, alpha_u, omega, sigma, score; };

// How a row's interval sums are to be read (RowStats::mode).
constexpr float kSumsFull = 0.f;         // all five sums
constexpr float kSumsWidthOnly = 1.f;    // the caps are known to be inactive; only sum gw, sum gw^2 were accumulated
constexpr float kSumsComplement = 2.f;   // caps inactive, every width above 1/2: q[1] = sum ec, q[3] = sum ec^2
constexpr float kSumsDirect = 3.f;       // all five sums, of p^l_i and p^u_i - p^l_i themselves (no row factor)
constexpr float kSumsFlatPending = 8.f;  // added to the above: a flat row that flatrow_kernel has still to redo

// The sums arrive shifted: s = { sum (gl - kl), sum (gw - kw), sum (gl - kl)^2, sum (gw - kw)^2,
// sum (gl - kl)(gw - kw) } over the V tokens of the row, where (kl, kw) are the values of one of the row's own
// tokens.  Sums and sums of squares taken about such a point lose at most a factor V of fp64's 1e-16 when the
// squared mean is subtracted, however small the spread is against the mean (a row of equal logits has spread 0
// and mean > 0: about the origin the difference of the two moments is rounding noise of relative size 1e-8
// after the square root, which Omega ~ V then multiplies).  Pass kl = kw = 0 for plain sums.
__device__ __forceinline__ RowScore finish_score(const double* s, double S, float mode, const RowArgs& A,
                                                 double kl, double kw)
{
    // p^l_i = Bc gl_i and p^u_i - p^l_i = Wc gw_i (tensor-radius mode: the per-token factors are already
    // inside gl and gw)
    const double V = (double)A.V;
    if (mode >= kSumsFlatPending) mode -= kSumsFlatPending;        // marked, not (yet) redone: the sums are valid as they are
    if (mode == kSumsComplement) {
        // s[1], s[3]: sums of (ec_i - kw) and its square, ec_i = 1 - delta_i:  Omega = V - sum ec,
        // Var(delta) = Var(ec), the latter taken among the small ec_i themselves instead of among numbers that
        // all round to 1
        RowScore o;
        o.alpha_l = 1.0; o.alpha_u = 1.0;
        o.omega = V - (s[1] + V * kw);
        o.sigma = sqrt(fmax(0.0, s[3] - s[1] * s[1] / V) / V);
        o.score = o.omega * o.sigma;
        return o;
    }
    const bool capless = mode == kSumsWidthOnly;
    const bool direct = mode == kSumsDirect;
    const double Bc = direct ? 1.0 : (A.radius ? 1.0 : A.b) / S, Wc = direct ? 1.0 : (A.radius ? 1.0 : A.a - A.b) / S;
    const double sum_gl = s[0] + V * kl, sum_gw = s[1] + V * kw;
    // S_l <= 1 <= S_u holds for every radius (p^l_i <= x_i <= p^u_i token by token); the computed sums carry ~1e-7
    // of fp32 token arithmetic and may land on the wrong side of 1 for a one-hot row, which a cap of exactly 1
    // would turn into a spurious scaling
    const double Sl = fmin(1.0, Bc * sum_gl), Su = fmax(1.0, Bc * sum_gl + Wc * sum_gw);
    RowScore o;
    o.alpha_l = 1.0; o.alpha_u = 1.0;
    if (A.normalize && !capless) {
        o.alpha_l = fmin(1.0, A.cap_lo / Sl);
        o.alpha_u = fmax(1.0, A.cap_hi / Su);
    }
    // delta_i = alpha_u p^u_i - alpha_l p^l_i = alpha_u w_i + (alpha_u - alpha_l) p^l_i = cw gw_i + cl gl_i:
    // both coefficients are >= 0, so Omega is a sum of non-negative terms; the spread is that of
    // delta_i - (cw kw + cl kl) = cw (gw_i - kw) + cl (gl_i - kl).
    const double cw = o.alpha_u * Wc, cl = (o.alpha_u - o.alpha_l) * Bc;
    o.omega = cw * sum_gw + (capless ? 0.0 : cl * sum_gl);
    const double T1 = cw * s[1] + cl * s[0];
    const double T2 = cw * cw * s[3] + 2.0 * cw * cl * s[4] + cl * cl * s[2];
    o.sigma = sqrt(fmax(0.0, T2 - T1 * T1 / V) / V);
    o.score = o.omega * o.sigma;
    return o;
}

// The accept test of a drafted token in the log domain, fp64 (Algorithm 1, "Cloud verification"):
//   ln p_x = cx - n ln2 - ln S,  ln q_x = tx - nt ln2 - ln Z;  accepted iff ln u < min(0, ln q_x - ln p_x).
// Returns whether the token is rejected.
template <typename T>
__device__ __forceinline__ bool reject_exact(float cx, float tx, float u, float n, float nt, double S, double Z)
{
    const double lp = ln_exp2<T>(cx, (double)n) - log(S);
    const double lq = ln_exp2<T>(tx, (double)nt) - log(Z);
    const double lnu = log((double)u);                             // log(0) = -inf: always accepted
    return !(lnu < fmin(0.0, lq - lp));
}

// The same test in fp32 with the hardware logarithm, for the streaming kernel, where every wave of a row evaluates
// it: 1 = accepted, 0 = rejected, -1 = too close to call (then reject_exact decides).  The fp32 evaluation is off by
// at most ~3e-7 (1 + the sum of the magnitudes of its terms): a hardware logarithm good to an ulp, a handful of
// roundings at 6e-8; the guard band is thirty times that, and a row falls inside it about once in a few thousand.
// Anything that is not a number ends up in the band.
__device__ __forceinline__ int accept_quick(float cx, float tx, float u, float n, float nt, float S, float Z)
{
    const float lS = __builtin_amdgcn_logf(S), lZ = __builtin_amdgcn_logf(Z);   // base 2
    const float lu = __builtin_amdgcn_logf(u);
    const float d = tx - cx, dn = nt - n;
    const float ell = fmaf(-(dn + (lZ - lS)), 0.693147181f, d);   // ln q_x - ln p_x
    const float margin = fminf(0.f, ell) - lu * 0.693147181f;     // > 0: accepted
    const float guard = 1e-5f * (1.f + fabsf(d) + fabsf(dn) + fabsf(lZ) + fabsf(lS) + fabsf(lu));
    if (u == 0.f && ell > -INFINITY) return 1;                     // ln 0 = -inf lies below every finite bound
    if (margin > guard) return 1;
    if (margin < -guard) return 0;
    return -1;
}

// One row's outputs from its statistics, in fp64 (Eq. uncertainty_score; Algorithm 1's threshold and verification
// steps): score, flag, the reported token's interval, the accept test in the log domain.  xid = the reported
// token (-1: the arg-max token, whose logit is st.mc), cx / tx / rawx = its centre logit, verifier logit and raw
// radius, u = the row's uniform for the accept test.  Returns whether the drafted token is rejected.
// T: the logits' type (the exponentials of its rows).  raw_top: tensor radius, rows with a token above 1/2: that token's raw radius.  flag: where the row's flag goes besides
// A.flags, if anywhere.  again(score): whether the row's sums are to be taken anew -- then nothing is written and the
// result is true.
struct NeverAgain { __device__ bool operator()(const RowScore&) const { return false; } };
template <typename T, bool RAD_TOP = false, typename Again = NeverAgain>
__device__ __forceinline__ bool finish_row(const RowArgs& A, int64_t row, const RowStats& st, float cx, float tx,
                                           float rawx, float u, bool do_q, bool do_v, float raw_top = 0.f,
                                           uint8_t* flag = nullptr, Again again = {})
{
    const double S = st.S;
    const float n = st.n;
    if (do_q) {
        double q[5] = {st.q[0], st.q[1], st.q[2], st.q[3], st.q[4]};
        // The token above 1/2 of a row whose caps can be active, once more in fp64.  Where a cap is active
        // Omega = alpha_u S_u - alpha_l S_l is a small difference of numbers near 1, and on a nearly one-hot row S_l is
        // little more than that token's lower bound: its fp32 evaluation in the streaming kernel (a hardware reciprocal
        // of a rounded product and three more roundings) leaves ~2e-7 of it, the whole absolute tolerance of an Omega of
        // 0.01 (a seeded random case: 2.04e-7 off).  At most one token of a row is above 1/2: the row's largest, whose
        // wave has the row's reference, so its e and the fp32 values that the scalar-radius pass has added to the sums
        // can be formed again here, by the same instructions, and exchanged for the fp64 values.  (Plain sums only:
        // such a row is not flat.  Wide scalar radii and tiny vocabularies come from other passes.)
        // With a radius tensor likewise (RAD_TOP: raw_top is that token's raw radius), from the fp32 radius: its error moves
        // the bounds by p (1 - p) times as much.  (A template parameter: one window in a tight loop waits for the kernel's
        // instructions to arrive as well.)
        // (the call's constants through an empty asm: what is derived from them here is otherwise formed at the top of
        // the calling kernel and kept -- in the streaming kernel: spilled -- through its row loop)
        double fa = A.a, fb = A.b;
        int fv = A.V;
        asm volatile("" : "+s"(fa), "+s"(fb), "+s"(fv));
        if (st.mode == kSumsFull && A.normalize && fv > kTinyVocab && (RAD_TOP || (!A.radius && fa < 3.0 * (double)fv)) &&
            st.kl == 0.0 && st.kw == 0.0) {
            const float etop = Elt<T>::exp2_ref(st.mc, n == -INFINITY ? 0.f : n);
            if ((double)etop > 0.5 * S) {
                const double ed = (double)etop, invS = 1.0 / S;
                const double x = ed * invS, om = fmax(0.0, S - ed) * invS;      // 1 - x from the sum of the other tokens
                double gl, gw, glf, gwf;
                if constexpr (RAD_TOP) {
                    const RadiusMode rm = radius_mode(A);
                    float plf, wf;
                    fuse_token_rad<T>(etop, raw_top, fuse_row_inv(recip(S), fa, fb), rm, plf, wf);
                    glf = (double)plf; gwf = (double)wf;
                    const double am1 = (double)(rm.unit ? radius_am1<T, true>(raw_top, rm.kappa, rm.rmax, rm.am1_max)
                                                        : radius_am1<T, false>(raw_top, rm.kappa, rm.rmax, rm.am1_max));
                    gl = ed / (1.0 + am1 * om);
                    gw = am1 * (am1 + 2.0) * om * gl / (1.0 + am1 * x);
                } else {
                    const double du = 1.0 + (fa - 1.0) * x, dl = fb + (1.0 - fb) * om;
                    gl = ed / dl; gw = gl * om / du;
                    float g, duf, omf;
                    fuse_parts<true>(etop, fuse_row_inv(recip(S), fa, fb), g, duf, omf);
                    glf = (double)(g * duf); gwf = (double)(g * omf);
                }
                q[0] += gl - glf;
                q[1] += gw - gwf;
                q[2] += gl * gl - glf * glf;
                q[3] += gw * gw - gwf * gwf;
                q[4] += gl * gw - glf * gwf;
            }
        }
        const RowScore rs = finish_score(q, S, st.mode, A, st.kl, st.kw);
        if (again(rs)) return true;
        if (A.omega) A.omega[row] = (float)rs.omega;
        if (A.sigma) A.sigma[row] = (float)rs.sigma;
        if (A.score) A.score[row] = (float)rs.score;
        if (A.flags) A.flags[row] = (uint8_t)(rs.score > A.tau);
        if (flag) *flag = (uint8_t)(rs.score > A.tau);
        if (A.p_lo || A.p_mid || A.p_hi) {
            // e_x exactly as the streaming kernel summed it into S (the arg-max token, the only one whose
            // probability can approach 1, sits in a wave whose reference is n), so that S - e_x is the
            // sum of the other tokens to fp64 rounding and 1 - x keeps its relative accuracy as x -> 1:
            // the lower bound's denominator b + (1-b)(1-x) is that small number when b is small too.
            const double ex = (double)Elt<T>::exp2_ref(cx, n == -INFINITY ? 0.f : n);
            const double x = ex / S, omx = fmax(0.0, S - ex) / S;
            double a = A.a, b = A.b;
            if (A.radius) {
                // the reported token's own radius (the launcher supplies ids in this mode)
                const double r = radius_of((double)rawx, A.kappa, A.rmax);
                a = exp(r); b = exp(-r);
            }
            if (A.p_mid) A.p_mid[row] = (float)x;
            if (A.p_lo) A.p_lo[row] = (float)(rs.alpha_l * b * x / (b + (1.0 - b) * omx));
            if (A.p_hi) A.p_hi[row] = (float)(rs.alpha_u * a * x / (1.0 + (a - 1.0) * x));
        }
    }
    bool rej = false;
    if (do_v) {
        rej = reject_exact<T>(cx, tx, u, n, st.nt, S, st.Z);
        if (A.accept) A.accept[row] = (uint8_t)(!rej);
        if (A.row_id && !rej) A.row_id[row] = -1;
    }
    return rej;
}

// The rows of a window that spans workgroups meet in one 64-bit word of caller memory, which needs no
// initialisation and carries everything the window's outputs need, so that no other memory has to be made visible
// between workgroups:  [63:33] the launch's tag (RowArgs::tag, never zero, different for every launch of the process: a
// word with another tag -- what an earlier call left behind, or whatever the memory held before -- is a fresh one),
// [32:25] rows arrived, [24:17] offset of the first rejected row so far (255: none), [16:0] that row's draw.
// A run of `rows` consecutive rows of the window that one workgroup has finished arrives with one call: its rows'
// first rejected offset in the window and that row's draw (id = -1: all accepted).  The call that completes the
// window returns true with the window's first rejected offset (-1: none) and its draw.
constexpr int kMaxCountedWindow = 32;                               // (the word would hold 255 rows)
__device__ __forceinline__ bool window_arrive(unsigned long long* p, uint32_t tag, int rows, int off, int id, int len,
                                              int& first, int& draw)
{
    const unsigned long long t31 = (unsigned long long)(tag & 0x7fffffffu);
    // The first exchange assumes a fresh word, which window_claim has normally left there at the start of the
    // kernel: the trip to memory and back that reading the word first would cost is the tail of the kernel.
    unsigned long long seen = (t31 << 33) | (0xffull << 17);
    for (;;) {
        const unsigned long long cur = (seen >> 33) == t31 ? seen : ((t31 << 33) | (0xffull << 17));
        const unsigned long long count = ((cur >> 25) & 0xffull) + (unsigned long long)rows;
        unsigned long long f = (cur >> 17) & 0xffull, d = cur & 0x1ffffull;
        if (id >= 0 && (unsigned long long)off < f) { f = (unsigned long long)off; d = (unsigned long long)id & 0x1ffffull; }
        const unsigned long long next = (t31 << 33) | (count << 25) | (f << 17) | d;
        const unsigned long long prev = atomicCAS(p, seen, next);
        if (prev == seen) {
            first = f == 0xffull ? -1 : (int)f;
            draw = (int)d;
            if (count != (unsigned long long)len) return false;
            // complete: hand the word back (a replay of this launch from a captured graph carries the same tag)
            __hip_atomic_store(p, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        }
        seen = prev;                                               // another row of the window got in between
    }
}

// Makes a window's word a fresh one of this launch ahead of its rows' arrivals (an optimisation only: window_arrive
// copes with whatever it finds).
// `seen` = what the caller has read in the word (an atomic load issued early, so that its trip to memory is over).
// One exchange whose outcome is not awaited: if it fails, another workgroup has claimed the word or arrived in it in
// the meantime, and the word is what it should be.
__device__ __forceinline__ void window_claim(unsigned long long* p, uint32_t tag, unsigned long long seen)
{
    const unsigned long long t31 = (unsigned long long)(tag & 0x7fffffffu), fresh = (t31 << 33) | (0xffull << 17);
    if ((seen >> 33) != t31) (void)atomicCAS(p, seen, fresh);
}

// Compute units of the current device (asked once per device, then cached; the cache is a relaxed atomic per device:
// two threads that ask at once both write the same number).
inline int compute_units()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    static std::atomic<int> cache[64];
    int cus = cache[dev].load(std::memory_order_relaxed);
    if (cus == 0) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        cache[dev].store(cus, std::memory_order_relaxed);
    }
    return cus;
}

// The grid of a kernel whose workgroups walk over `pieces` pieces of work and have room for at most `most` of them each:
// one workgroup per piece, else as many as are resident at a time, or that several times over (taking their turn) -- whole
// rounds, so that the last one leaves no compute unit idle.  (The fewest workgroups that hold the pieces may be a few more
// than are resident: those few then run alone.  With one workgroup to a unit, fused 33000 x 65536 bf16 3553 -> 2053 us, three
// heads' Ensemble 9000 x 16384 bf16 969 -> 561, the loss 20000 x 16384 fp32 1355 -> 882; with sixteen, where the first to
// end make room for the last, the quantifier with a radius tensor 80000 x 1024 fp32 156 -> 142.)
inline int64_t whole_rounds(int64_t pieces, int64_t most, int64_t resident)
{
    const int64_t g = resident * ((pieces + resident * most - 1) / (resident * most));
    return g < pieces ? g : pieces;
}

}  // namespace
}  // namespace ciar
