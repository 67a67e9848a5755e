// gfx950 (MI355X, CDNA4) kernels of the Quantized-Adam-with-error-feedback step
// (arXiv 2004.14180: Sec. 5.1 for the quantizers Q_g and Q_x, Algorithm 1 for the
// moments / step / residual, Algorithm 2 (gather step) for the mean over workers).
//
// Everything here is a streaming pass bound by HBM bandwidth: no contraction, no MFMA.  The design
// rules are the ones that matter for that regime on CDNA4:
//   * 64-wide wavefronts; a lane owns 4 consecutive fp32 values so every global access is a 128-bit
//     load/store and a wavefront touches 1 KiB of contiguous memory;
//     all buffers are touched once per pass, so loads and stores carry the non-temporal hint, except where the next
//     pass finds the data in the memory-side cache (keep_scanned, keep_parked);
//   * work is cut along tiles (<= 4096 elements of one layer), so all per-layer quantities (scales, code
//     offsets) are wave-uniform and live in scalar registers;
//   * the scale pass and variant W's first pass run as 256-thread workgroups; the main pass, both quantizers and
//     the server as workgroups of ONE wavefront each, which drift apart and so mix their reads and writes (see
//     Items); the loads of a group of workers are issued together before any arithmetic;
//   * the per-layer scale is a max over |g+e|: lanes reduce with integer max on the bit pattern
//     (non-negative floats order like integers; NaN/Inf sort above every finite value and so
//     surface in the scale), wavefront reduction by cross-lane shuffles, LDS across the four
//     wavefronts, one plain store of the tile's maximum; the tile maxima of a layer are folded by a
//     second small kernel, or where they are few by the quantizing wavefronts themselves.  No atomics in these
//     passes: thousands of workgroups hitting one freshly zeroed word at the start of every layer cost more than the whole
//     pass (the workgroups of k_parked, which are few per layer, count themselves with one each);
//   * a segment that starts off the 16-byte grid keeps the same lane-to-element mapping (the codes are
//     anchored at the segment start) and moves its data with dword-aligned 128-bit accesses;
//   * layers of up to 17.8 M elements in long lists stay on the chip between the scale and the quantizer: the workgroups of a
//     layer meet over its scale while they load and store units of other layers (k_parked);
//   * when the error buffers are what the previous step wrote, |e| <= s/4 (half the widest gap of
//     the grid), so an element whose |g| lies that far below a known lower bound of the scale
//     cannot be the maximum: the filtered scale pass takes the exact maxima of every 64th tile as
//     that lower bound and then reads g alone, and e only for the few elements that can matter;
//   * codes are stored as bit planes of 32-element groups; a lane's four codes are combined with
//     the other seven lanes of its group by three DPP OR steps per plane, so packing costs no
//     LDS traffic and no scatter;
//   * fp32 arithmetic is kept bit-reproducible: one rounding per operation (built with
//     -ffp-contract=off), IEEE division and square root, subnormals kept.  The quotient p/s that
//     selects the grid level is taken as p * (1/s) and redone with the IEEE division only when it
//     lands within 8 ulp of a decision threshold, which cannot change any decision (the product
//     is within 2.5 ulp of the correctly rounded quotient).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>
#include <type_traits>

#include "qadam_internal.h"

namespace qadam {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t f2u(float f) { return __float_as_uint(f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __uint_as_float(u); }

// ------------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): counter (c0..c3), key (k0,k1) -> four 32-bit words.  HALVES: the products' halves by a
// multiplication each, else both by one.  us, halves / one: the main pass, whose registers the 64-bit products crowd, one worker
// of 20 M (2^20) elements 177 / 199, 4.7 M 51.1 / 52.8, four of 20 M 375 / 378; k_parked, GPT-2 small, 8 workers 3419 / 3382 per
// step, off the grid 4088 / 3925; worker quantizer off the grid, 80 M 303 / 287; weight quantizer, 5 M 13.1 / 12.7.
// ------------------------------------------------------------------------------------------------
template <bool HALVES>
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint32_t hi0, lo0, hi1, lo1;
        if constexpr (HALVES) {
            hi0 = __umulhi(M0, c0); lo0 = M0 * c0;
            hi1 = __umulhi(M1, c2); lo1 = M1 * c2;
        } else {
            const uint64_t m0 = (uint64_t)M0 * c0, m1 = (uint64_t)M1 * c2;
            hi0 = (uint32_t)(m0 >> 32); lo0 = (uint32_t)m0;
            hi1 = (uint32_t)(m1 >> 32); lo1 = (uint32_t)m1;
        }
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += W0;
        k1 += W1;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Uniforms in [0,1) with 24 bits for the V consecutive elements starting at global index gi.
// Counter = (gi/4 low, gi/4 high, step, worker + (stream << 16)); element j takes word j mod 4.
template <int V, bool HALVES>
__device__ __forceinline__ void uniforms(const StepScalars& S, int64_t gi, uint32_t worker, uint32_t stream,
                                         float (&U)[V])
{
    const uint64_t blk = (uint64_t)gi >> 2;
    uint32_t out[4];
    philox4x32_10<HALVES>((uint32_t)blk, (uint32_t)(blk >> 32), S.step, worker + (stream << 16), S.key0, S.key1, out);
    if constexpr (V == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) U[j] = (float)(out[j] >> 8) * 0x1p-24f;
    } else {
        const int wsel = (int)(gi & 3);
        const uint32_t w = wsel == 0 ? out[0] : wsel == 1 ? out[1] : wsel == 2 ? out[2] : out[3];
        U[0] = (float)(w >> 8) * 0x1p-24f;
    }
}

// ------------------------------------------------------------------------------------------------
// Q_g on one value (Sec. 5.1).  r = p / s lies in [-1, 1]; the grid is {0} and 2^(mu-1-k_g),
// mu = 1..k_g+1.  Nearest point: the midpoint below level 2^-j is 0.75 * 2^-j, i.e. mantissa
// 0x400000 one exponent lower, so adding 0x400000 to the bit pattern of |r| and keeping the
// exponent field rounds |r| to the nearest power of two with midpoints going up.  Below the first
// level 2^-k_g the only midpoint is 2^(-k_g-1) (halfway to zero).
// ------------------------------------------------------------------------------------------------
struct QgConst {
    int ebias;             // 126 - k_g: exponent field of level mu is mu + ebias
    uint32_t half_l1_bits; // bit pattern of 2^(-k_g-1)
    uint32_t l1_bits;      // bit pattern of 2^-k_g
    float up, down;        // 2^(k_g+2) and its reciprocal: a level times `up` is 2^(mu+1)
};

__device__ __forceinline__ QgConst make_qg(int k_g)
{
    QgConst c;
    c.ebias = 126 - k_g;
    c.half_l1_bits = (uint32_t)(126 - k_g) << 23;
    c.l1_bits = (uint32_t)(127 - k_g) << 23;
    c.up = u2f((uint32_t)(129 + k_g) << 23);
    c.down = u2f((uint32_t)(125 - k_g) << 23);
    return c;
}

// bit pattern of the grid point nearest to |r| (0 for the zero level); `zero_below` is
// half_l1_bits, or 0xffffffff to force every level to zero (invalid scale)
__device__ __forceinline__ uint32_t qg_nearest_bits(uint32_t ab, const QgConst& c, uint32_t zero_below)
{
    uint32_t lvl = (ab + 0x00400000u) & 0x7f800000u;
    lvl = lvl > c.l1_bits ? lvl : c.l1_bits;
    lvl = lvl < 0x3f800000u ? lvl : 0x3f800000u;
    return ab >= zero_below ? lvl : 0u;
}

// unbiased choice between the neighbours lo <= |r| < hi: up with probability (|r|-lo)/(hi-lo)
__device__ __forceinline__ uint32_t qg_stochastic_bits(uint32_t ab, const QgConst& c, float U, bool valid)
{
    if (ab >= 0x3f800000u) return valid ? 0x3f800000u : 0u;
    uint32_t lo = ab & 0x7f800000u;                         // largest power of two <= |r|
    lo = lo >= c.l1_bits ? lo : 0u;                         // below the first level the lower neighbour is 0
    const uint32_t width = lo ? lo : c.l1_bits;             // hi - lo, a power of two
    const float inv_width = u2f((254u << 23) - width);      // exact reciprocal
    const float frac = (u2f(ab) - u2f(lo)) * inv_width;
    const uint32_t hi = lo ? lo + (1u << 23) : c.l1_bits;
    const uint32_t lvl = U < frac ? hi : lo;
    return valid ? lvl : 0u;
}

// The four codes of a lane from its levels times 2^(k_g+2), with the sign of p: +-2^(mu+1), whose exponent field is 128 + mu, or
// +-0.  Element j's code is the four bits from bit 0, 16, 4 and 20 on (spread so that pack_planes gathers a plane's four bits
// with one multiplication).
__device__ __forceinline__ uint32_t pack_codes(const uint32_t (&L)[4], int mu_bits)
{
    uint32_t half[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t h = __builtin_amdgcn_perm(L[2 * k + 1], L[2 * k], 0x07060302u);     // the upper halves of two of them
        const uint32_t sign = h & (h << 1) & 0x80008000u;                                   // no sign for the level 0
        half[k] = (h & 0x03800380u) | (sign >> (8 - mu_bits));
    }
    return half[0] >> 7 | half[1] >> 3;
}

// One worker's share of one lane, p = g + e: level, dequantized value q, which is added to acc, residual p - q, and the
// lane's codes (pack_codes).  s is the layer scale, inv_s its reciprocal or 0 when the fast quotient must not be used (tiny,
// huge, zero or non-finite scale).
// The fast form works on p / s times 2^(k_g+2), where the levels are 4, 8, .. and what is below 2 goes to 0, whatever k_g.
// Products with these powers of two and with the levels are exact for the scales it is used with, so that the sums with one
// rounding, p - s L and acc + s L, are what a multiplication and an addition give; the level 0 takes the sign -0, whose product
// leaves both of them as they are and makes a residual of +0 of p = -0, as p - q does.
// Bound by the vector ALUs where few wavefronts share a SIMD.  97 vector instructions for four
// elements and their three planes, 138 with the levels' own exponents, a multiplication and an addition each and codes put
// together one by one.  us per step, that way / this way: 10 k elements in one workgroup 5.89 / 5.21; 11.7 M
// parameters, 4 workers 195.4 / 190.5; GPT-2 small, 4 workers by separate calls 2078 / 2059.
template <int ROUNDING>
__device__ __forceinline__ void worker_lane(const float (&p)[4], float s, float inv_s, const QgConst& c, int mu_bits,
                                            const float (&U)[4], float (&acc)[4], float (&enew)[4], uint32_t& codes)
{
    float r[4];
    uint32_t L[4];
    if (ROUNDING == 0 && inv_s != 0.0f) {
        const float inv_up = inv_s * c.up, s_down = s * c.down;
        uint32_t near = 0xffffffffu;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            r[j] = p[j] * inv_up;
            // within 8 ulp of a power of two or of 0.75 times one?
            near = min(near, (f2u(r[j]) + 8u) << 10);
        }
        if (near < 16u << 10) {
#pragma unroll
            for (int j = 0; j < 4; ++j) r[j] = (p[j] / s) * c.up;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // as qg_nearest_bits, 2^(k_g+2) times as large
            const float lvl = __builtin_amdgcn_fmed3f(u2f((f2u(r[j]) + 0x00400000u) & 0x7f800000u), 4.0f, c.up);
            L[j] = fabsf(r[j]) >= 2.0f ? f2u(copysignf(lvl, r[j])) : 0x80000000u;
            acc[j] = __builtin_fmaf(s_down, u2f(L[j]), acc[j]);
            enew[j] = __builtin_fmaf(-s_down, u2f(L[j]), p[j]);
        }
    } else {
        const bool valid = s > 0.0f && s < __builtin_inff();
        const uint32_t zero_below = valid ? c.half_l1_bits : 0xffffffffu;
        const float s_mul = valid ? s : 0.0f;               // an invalid scale quantizes everything to 0
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = p[j] / s;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t ab = f2u(r[j]) & 0x7fffffffu, sign = f2u(p[j]) & 0x80000000u;
            uint32_t lvl;
            if constexpr (ROUNDING == 0) lvl = qg_nearest_bits(ab, c, zero_below);
            else lvl = qg_stochastic_bits(ab, c, U[j], valid);
            const float qa = s_mul * u2f(lvl);                // s * 2^(mu-1-k_g); 0 when lvl == 0
            const float qv = u2f(f2u(qa) | sign);
            acc[j] = acc[j] + qv;
            enew[j] = p[j] - qv;
            L[j] = f2u(u2f(lvl) * c.up) | sign;
        }
    }
    codes = pack_codes(L, mu_bits);
}

// Value of the code stored at bit `pos` of a 32-element group's plane words w[0..MU_BITS]
// (planes 0..MU_BITS-1 hold the level index mu, plane MU_BITS the sign), with layer scale s:
// +-s * 2^(mu-1-k_g), or 0 for mu == 0.  The bits are taken straight from the words, so no
// per-element code has to be assembled first.
template <int MU_BITS>
__device__ __forceinline__ float qg_decode_planes(const uint32_t (&w)[4], uint32_t pos, float s, const QgConst& c)
{
    uint32_t mu = __builtin_amdgcn_ubfe(w[0], pos, 1u);
#pragma unroll
    for (int k = 1; k < MU_BITS; ++k) mu |= __builtin_amdgcn_ubfe(w[k], pos, 1u) << k;
    const uint32_t sign = (w[MU_BITS] << (31u - pos)) & 0x80000000u;
    const float lvl = u2f((mu + (uint32_t)c.ebias) << 23);
    float qa = s * lvl;
    qa = mu > 0u ? qa : 0.0f;
    return u2f(f2u(qa) | sign);
}

// Four consecutive elements of a lane at once, added to acc: q_j = s * L_j with L_j = +-2^(mu-1-k_g) or 0, which binary16
// holds in its upper byte.  The plane bits of the four elements are spread to the four bytes of a word, one byte permute
// looks the four levels up, and since s * L_j is exact for the scales this is used with (fast_scale), the sum with one
// rounding, acc + s * L_j, is what a multiplication and an addition give.  18 vector instructions for four elements of 3-bit
// codes where bit by bit it is 40.
struct Levels {
    uint32_t lo, hi;       // byte mu: upper byte of binary16 2^(mu-1-k_g), mu = 0..3 and 4..7
};

__device__ __forceinline__ Levels make_levels(int k_g)
{
    uint64_t b = 0;
#pragma unroll
    for (int mu = 1; mu < 8; ++mu) b |= (uint64_t)((14 + mu - k_g) << 2) << (8 * mu);
    return {(uint32_t)b, (uint32_t)(b >> 32)};
}

__device__ __forceinline__ uint32_t spread4(uint32_t word, uint32_t pos)
{
    return __umul24(__builtin_amdgcn_ubfe(word, pos, 4u), 0x204081u) & 0x01010101u;
}

template <int MU_BITS>
__device__ __forceinline__ void add_decoded(const uint32_t (&w)[4], uint32_t pos, float s, const Levels& T, float (&acc)[4])
{
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    uint32_t mu = spread4(w[0], pos);
#pragma unroll
    for (int k = 1; k < MU_BITS; ++k) mu |= spread4(w[k], pos) << k;
    const uint32_t l = __builtin_amdgcn_perm(T.hi, T.lo, mu) | (spread4(w[MU_BITS], pos) << 7);
    const h2 a = __builtin_bit_cast(h2, __builtin_amdgcn_perm(0u, l, 0x010c000cu));
    const h2 b = __builtin_bit_cast(h2, __builtin_amdgcn_perm(0u, l, 0x030c020cu));
    acc[0] = __builtin_fmaf((float)a.x, s, acc[0]);
    acc[1] = __builtin_fmaf((float)a.y, s, acc[1]);
    acc[2] = __builtin_fmaf((float)b.x, s, acc[2]);
    acc[3] = __builtin_fmaf((float)b.y, s, acc[3]);
}

// scales from 2^-100 to 2^100: s * 2^-6 .. s * 2^6 are normal numbers
__device__ __forceinline__ bool fast_scale(float s) { return f2u(s) - (27u << 23) <= (200u << 23); }

// ------------------------------------------------------------------------------------------------
// Bit-plane packing.  A lane holds the codes of elements 4*lane..4*lane+3 of a 256-element
// wave chunk as pack_codes leaves them; the 8 lanes 8G..8G+7 form 32-element group G.  For plane k
// every lane gathers its 4 plane bits (a multiply moves bits 0,16,4,20 to bits 17..20), shifts them
// to position 4*(lane%8) and the group ORs them with three DPP steps (swap within pairs, swap
// pairs within quads, mirror the two quads of a half row).  Lane 8G+k keeps word k.  Must be
// called with all 64 lanes active.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t dpp_or8(uint32_t w)
{
    w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    w |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x141, 0xF, 0xF, false);  // row_half_mirror
    return w;
}

__device__ __forceinline__ uint32_t pack_planes(uint32_t codes, int code_bits, int lane, int& word_slot, bool& writes)
{
    uint32_t sel = 0;
    const int sub = lane & 7;
    const int sh = sub * 4;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k < code_bits) {
            const uint32_t t = codes & (0x00110011u << k);
            const uint32_t nib = (__umul24(t, 0x28005u) >> (17 + k)) & 0xFu;
            const uint32_t w = dpp_or8(nib << sh);
            sel = sub == k ? w : sel;
        }
    }
    word_slot = (lane >> 3) * code_bits + sub;     // word within the wave chunk's 8 groups
    writes = sub < code_bits;
    return sel;
}

// plane words of the 32-element group that holds this lane's V elements, and the bit position of
// the lane's first element in them (inverse of pack_planes)
template <int V, int MU_BITS>
__device__ __forceinline__ uint32_t load_planes(const uint32_t* __restrict__ chunk_words, int lane, uint32_t (&w)[4])
{
    constexpr int CODE_BITS = MU_BITS + 1;
    static_assert(V == 4, "a lane owns four consecutive elements");
    const uint32_t* gw = chunk_words + (lane >> 3) * CODE_BITS;
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = k < CODE_BITS ? gw[k] : 0u;
    return (uint32_t)(lane & 7) * 4u;
}

// ------------------------------------------------------------------------------------------------
// guarded vector access: one 128-bit non-temporal access when the lane's V=4 elements are all
// inside the tile (every buffer is streamed exactly once per pass)
// ------------------------------------------------------------------------------------------------
template <int V>
__device__ __forceinline__ void load_v(const float* __restrict__ p, int nvalid, float (&out)[V])
{
    if constexpr (V == 4) {
        if (nvalid == 4) {
            const f4 t = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
            out[0] = t.x; out[1] = t.y; out[2] = t.z; out[3] = t.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) out[j] = j < nvalid ? p[j] : 0.0f;
        }
    } else {
        out[0] = nvalid > 0 ? p[0] : 0.0f;
    }
}

template <int V>
__device__ __forceinline__ void store_v(float* __restrict__ p, int nvalid, const float (&in)[V])
{
    if constexpr (V == 4) {
        if (nvalid == 4) {
            f4 t;
            t.x = in[0]; t.y = in[1]; t.z = in[2]; t.w = in[3];
            __builtin_nontemporal_store(t, reinterpret_cast<f4*>(p));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) if (j < nvalid) p[j] = in[j];
        }
    } else {
        if (nvalid > 0) p[0] = in[0];
    }
}

template <int V>
__device__ __forceinline__ void store_wcodes(void* __restrict__ base, int wcode_bytes, int64_t gi, int nvalid,
                                             const int (&j)[V])
{
    if (wcode_bytes == 1) {
        int8_t* p = static_cast<int8_t*>(base) + gi;
        if constexpr (V == 4) {
            if (nvalid == 4) {
                const uint32_t packed = ((uint32_t)j[0] & 0xFFu) | (((uint32_t)j[1] & 0xFFu) << 8) |
                                        (((uint32_t)j[2] & 0xFFu) << 16) | ((uint32_t)j[3] << 24);
                __builtin_nontemporal_store(packed, reinterpret_cast<uint32_t*>(p));
                return;
            }
        }
#pragma unroll
        for (int t = 0; t < V; ++t) if (t < nvalid) p[t] = (int8_t)j[t];
    } else {
        int16_t* p = static_cast<int16_t*>(base) + gi;
        if constexpr (V == 4) {
            if (nvalid == 4) {
                s4 t;
                t.x = (short)j[0]; t.y = (short)j[1]; t.z = (short)j[2]; t.w = (short)j[3];
                __builtin_nontemporal_store(t, reinterpret_cast<s4*>(p));
                return;
            }
        }
#pragma unroll
        for (int t = 0; t < V; ++t) if (t < nvalid) p[t] = (int16_t)j[t];
    }
}

// ------------------------------------------------------------------------------------------------
// Tiles of a segment that does not start on a 16-byte boundary.  The packed codes are anchored at the
// segment start (a lane's four elements are four consecutive bits of a plane word), so a lane's four
// values lie r = (flat start mod 4) floats off the 16-byte grid of memory.  The lane still moves them
// with ONE 128-bit access: the vector type below carries 4-byte alignment, for which the compiler emits
// the same global_load/store_dwordx4 (the memory unit of this target accepts dword-aligned wide
// accesses); a wavefront's access is still one contiguous 1 KiB run, it merely touches nine 128-byte
// lines instead of eight.  The weight codes (four int8 or int16) are stored likewise through types of
// element alignment.  What differs besides is the random stream of stochastic rounding, which is
// indexed by the flat element number (below).
// ------------------------------------------------------------------------------------------------
typedef f4 f4_a4 __attribute__((aligned(4)));
typedef uint32_t u32_a1 __attribute__((aligned(1)));
typedef s4 s4_a2 __attribute__((aligned(2)));

struct Shift {
    int r;              // flat index of the tile's first element mod 4 (1..3 when used)
};

__device__ __forceinline__ Shift make_shift(const Tile& t)
{
    Shift sf;
    sf.r = (int)(t.start & 3);
    return sf;
}

__device__ __forceinline__ void load_shifted(const float* __restrict__ p, int nvalid, float (&out)[4])
{
    if (nvalid == 4) {
        const f4 t = *reinterpret_cast<const f4_a4*>(p);
        out[0] = t.x; out[1] = t.y; out[2] = t.z; out[3] = t.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = j < nvalid ? p[j] : 0.0f;
    }
}

// wherever it lies
__device__ __forceinline__ void load_any(const float* __restrict__ p, int nvalid, float (&out)[4])
{
    if (nvalid == 4) {
        const f4 t = __builtin_nontemporal_load(reinterpret_cast<const f4_a4*>(p));
        out[0] = t.x; out[1] = t.y; out[2] = t.z; out[3] = t.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = j < nvalid ? p[j] : 0.0f;
    }
}

__device__ __forceinline__ void store_shifted(float* __restrict__ p, int nvalid, const float (&in)[4])
{
    if (nvalid == 4) {
        f4 t;
        t.x = in[0]; t.y = in[1]; t.z = in[2]; t.w = in[3];
        __builtin_nontemporal_store(t, reinterpret_cast<f4_a4*>(p));
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) if (j < nvalid) p[j] = in[j];
    }
}

// weight codes of the lane's four elements at element index gi (not a multiple of 4)
__device__ __forceinline__ void store_wcodes_shifted(void* __restrict__ base, int wcode_bytes, int64_t gi, int nvalid,
                                                     const int (&j)[4])
{
    if (wcode_bytes == 1) {
        int8_t* p = static_cast<int8_t*>(base) + gi;
        if (nvalid == 4) {
            const uint32_t packed = ((uint32_t)j[0] & 0xFFu) | (((uint32_t)j[1] & 0xFFu) << 8) |
                                    (((uint32_t)j[2] & 0xFFu) << 16) | ((uint32_t)j[3] << 24);
            __builtin_nontemporal_store(packed, reinterpret_cast<u32_a1*>(p));
            return;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) if (t < nvalid) p[t] = (int8_t)j[t];
    } else {
        int16_t* p = static_cast<int16_t*>(base) + gi;
        if (nvalid == 4) {
            s4 t;
            t.x = (short)j[0]; t.y = (short)j[1]; t.z = (short)j[2]; t.w = (short)j[3];
            __builtin_nontemporal_store(t, reinterpret_cast<s4_a2*>(p));
            return;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) if (t < nvalid) p[t] = (int16_t)j[t];
    }
}

// uniforms of four consecutive elements that start r into a Philox block: words r..3 of the block
// of gi and words 0..r-1 of the next one
template <bool HALVES>
__device__ __forceinline__ void uniforms_shifted(const StepScalars& S, int64_t gi, uint32_t worker, uint32_t stream,
                                                 int r, float (&U)[4])
{
    float lo[4], hi[4];
    uniforms<4, HALVES>(S, gi - r, worker, stream, lo);
    uniforms<4, HALVES>(S, gi - r + 4, worker, stream, hi);
    const bool r1 = r == 1, r2 = r == 2;
    U[0] = r1 ? lo[1] : (r2 ? lo[2] : lo[3]);
    U[1] = r1 ? lo[2] : (r2 ? lo[3] : hi[0]);
    U[2] = r1 ? lo[3] : (r2 ? hi[0] : hi[1]);
    U[3] = r1 ? hi[0] : (r2 ? hi[1] : hi[2]);
}

// the accessors of the tile loops: SH selects the shifted forms
template <int V, bool SH>
__device__ __forceinline__ void ld(const float* __restrict__ buf, int64_t gi, int nvalid, const Shift& sf, float (&out)[V])
{
    if constexpr (SH) load_shifted(buf + gi, nvalid, out);
    else load_v<V>(buf + gi, nvalid, out);
}

template <int V, bool SH>
__device__ __forceinline__ void st(float* __restrict__ buf, int64_t gi, int nvalid, const Shift& sf, const float (&in)[V])
{
    if constexpr (SH) store_shifted(buf + gi, nvalid, in);
    else store_v<V>(buf + gi, nvalid, in);
}

template <int V, bool SH>
__device__ __forceinline__ void stw(void* __restrict__ base, int wcode_bytes, int64_t gi, int nvalid, const Shift& sf,
                                    const int (&j)[V])
{
    if constexpr (SH) store_wcodes_shifted(base, wcode_bytes, gi, nvalid, j);
    else store_wcodes<V>(base, wcode_bytes, gi, nvalid, j);
}

template <int V, bool SH, bool HALVES = false>
__device__ __forceinline__ void unif(const StepScalars& S, int64_t gi, uint32_t worker, uint32_t stream, const Shift& sf,
                                     float (&U)[V])
{
    if constexpr (SH) uniforms_shifted<HALVES>(S, gi, worker, stream, sf.r, U);
    else uniforms<V, HALVES>(S, gi, worker, stream, U);
}

// ------------------------------------------------------------------------------------------------
// Server arithmetic on one lane: moments (Alg. 1, moment recursions) and the step alpha m / sqrt(v + eps).
// ------------------------------------------------------------------------------------------------
// of moments that have taken the step
__device__ __forceinline__ float adam_quotient(const StepScalars& S, float m, float v)
{
    if (S.adam_flavor == 0) {
        const float den = sqrtf(v + S.eps);
        return (S.lr * m) / den;
    } else {
        const float den = (sqrtf(v) / S.sbc2) + S.eps;
        return (S.lr1 * m) / den;
    }
}

__device__ __forceinline__ float adam_step(const StepScalars& S, float gbar, float& m, float& v)
{
    const float g2 = gbar * gbar;
    const float vn = (S.beta2 * v) + (S.omb2 * g2);
    const float mn = (S.beta1 * m) + (S.omb1 * gbar);
    v = vn;
    m = mn;
    return adam_quotient(S, mn, vn);
}

__device__ __forceinline__ float mean_over_workers(const StepScalars& S, float acc)
{
    // N a power of two: multiplying by the exact 1/N rounds exactly like dividing by N
    return S.n_is_pow2 ? acc * S.inv_n : acc / S.n_workers_f;
}

// Q_x on one value (Sec. 5.1): nearest multiple of 2^-(k_x+1), saturated to [-1/2, 1/2].
template <int ROUNDING>
__device__ __forceinline__ void qx_value(float y, float two_kx1, float inv_two_kx1, float jmax, float U,
                                         int& j, float& xhat)
{
    const float u = y * two_kx1;
    float jf;
    if constexpr (ROUNDING == 0) {
        const float t = truncf(u);
        const float d = fabsf(u - t);                   // exact
        jf = d >= 0.5f ? t + copysignf(1.0f, u) : t;     // halves away from zero
    } else {
        jf = floorf(u + U);
    }
    jf = fminf(fmaxf(jf, -jmax), jmax);
    jf = (u != u) ? 0.0f : jf;
    j = (int)jf;
    xhat = jf * inv_two_kx1;
}

template <int V, int ROUNDING, bool SH = false, bool HALVES = false>
__device__ __forceinline__ void weight_lane(const StepScalars& S, const float (&x)[V], const float (&werr_in)[V],
                                            int64_t gi, const Shift& sf, float (&werr_out)[V], int (&j)[V])
{
    const float two_kx1 = u2f((uint32_t)(127 + S.k_x + 1) << 23);
    const float inv = u2f((uint32_t)(127 - S.k_x - 1) << 23);
    const float jmax = u2f((uint32_t)(127 + S.k_x) << 23);
    float U[V];
#pragma unroll
    for (int t = 0; t < V; ++t) U[t] = 0.0f;
    if constexpr (ROUNDING == 1) unif<V, SH, HALVES>(S, gi, 0u, 1u, sf, U);
#pragma unroll
    for (int t = 0; t < V; ++t) {
        const float y = S.weight_ef ? x[t] + werr_in[t] : x[t];
        float xh;
        qx_value<ROUNDING>(y, two_kx1, inv, jmax, U[t], j[t], xh);
        werr_out[t] = y - xh;
    }
}

// ------------------------------------------------------------------------------------------------
// kernel argument blocks
// ------------------------------------------------------------------------------------------------
// the item of this workgroup (see Items)
__device__ __forceinline__ uint32_t wave_item(const Items& I) { return item_of(I, blockIdx.x); }

struct AmaxArgs {
    const Tile* tiles;
    int num_tiles;
    Items items;            // k_amax<true>: one tile each
    const float* grad[QADAM_MAX_WORKERS];
    const float* err[QADAM_MAX_WORKERS];
    uint32_t* tile_max;     // rows of `row` maxima, one row per worker
    int row;
    int first_worker;
    const int32_t* tile_list;   // null: workgroup b takes tile b; else tile tile_list[b] (the sampled tiles)
    const uint32_t* thr;        // filtered pass only: [N][L] thresholds on |g| as bit patterns (0: read everything)
    int num_segments;
    const float* err_bound;     // verification only: [N][L] bounds the error buffers must respect
    uint32_t* status;
    int64_t seg_len;            // tiles == null only: length of the single segment
};

// How a quantizing kernel comes by the scales.  tile_max == null: k_reduce_scales has written scales and reciprocals.
// Else every wavefront folds the maxima of its layer itself, and the first one of the layer writes out what
// k_reduce_scales would have written.
struct Fold {
    const uint32_t* tile_max;       // rows of `row` maxima, `per_tile` to a tile
    const int32_t* seg_tile_begin;  // null: one segment that owns the whole row
    int row, per_tile;
    int num_segments;
    float* inv_scales;              // [N][L]
    float* err_bound;               // [N][L]
    float bound_factor;
};

struct FusedArgs {
    const Tile* tiles;
    Items items;
    uint32_t* status;
    Fold fold;
    StepScalars S;
    ServerPtrs sp;
    const float* grad[QADAM_MAX_WORKERS];
    float* err[QADAM_MAX_WORKERS];
    uint32_t* codes[QADAM_MAX_WORKERS];
    float* scales[QADAM_MAX_WORKERS];
};

struct WorkerArgs {        // one worker
    const Tile* tiles;
    Items items;
    uint32_t* status;
    StepScalars S;
    const float* grad;     // variant S: g;  variant W second pass: null (p was parked in err)
    float* err;
    uint32_t* codes;
    float* scales;
    Fold fold;                 // its tables start at this worker's rows
    int worker;
    int64_t seg_len;           // tiles == null only: length of the single segment
};

// Tile record of workgroup `ti`: from the handle's table, or, for the handle-free single-segment
// call (tiles == null), computed from the segment length: tile ti covers elements
// [ti * kTileElems, ...) of a segment that starts 16-byte aligned at element 0.
__device__ __forceinline__ Tile tile_at(const Tile* __restrict__ tiles, int ti, int64_t seg_len, int code_bits)
{
    if (tiles) return tiles[ti];
    Tile t;
    t.start = (int64_t)ti * kTileElems;
    t.code_word = (int64_t)ti * (kTileElems / 32) * code_bits;
    const int64_t left = seg_len - t.start;
    t.len = (int32_t)(left < kTileElems ? left : kTileElems);
    t.seg = 0;
    t.flags = 0;
    if (left <= kTileElems) {
        const int64_t used = (seg_len + 31) / 32 * code_bits;
        t.flags = (int32_t)((used + 3) / 4 * 4 - used) << 8;     // zero words up to a multiple of 16 bytes
    }
    t.reserved = 0;
    return t;
}

struct ScaleArgs {
    float* scales[QADAM_MAX_WORKERS];
    float* inv_scales;
    const uint32_t* tile_max;
    const int32_t* seg_tile_begin;
    const int32_t* layers;  // null: all
    int first_worker, num_layers, num_segments, num_tiles;
    int row;                // maxima from one worker's to the next's
    int max_per_tile;       // maxima the pass before left per tile
    float* err_bound;       // [N][L]: bound on |e'| after the step that uses these scales
    uint32_t* thr;          // [N][L]: thresholds of the filtered pass (written by k_reduce_lower_bounds)
    float bound_factor;     // |e'| <= bound_factor * s for this quantizer and rounding mode
    int sample_stride;      // every sample_stride-th tile of a layer is a sampled tile
};

// ------------------------------------------------------------------------------------------------
// scales: per-tile max |g + e| (k_amax), then per (worker, layer) the max over the layer's tiles
// and its reciprocal for the fast quotient (k_reduce_scales)
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)v, d, 64);
        v = o > v ? o : v;
    }
    return v;
}

// block-wide max of the lanes' values; every thread gets the result
template <int THREADS = kBlockThreads>
__device__ __forceinline__ uint32_t block_max(uint32_t local)
{
    __shared__ uint32_t wave_part[THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t wm = wave_max_u32(local);
    if (lane == 0) wave_part[wave] = wm;
    __syncthreads();
    uint32_t bm = wave_part[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) bm = wave_part[w] > bm ? wave_part[w] : bm;
    return bm;
}

// load_v of the scale pass.  KEEP: an ordinary load, so that the lines stay in the 256 MB cache in front of the memory
// for the pass that quantizes them (keep_scanned says when); else the non-temporal one, which leaves no copy behind.
template <int V, bool KEEP>
__device__ __forceinline__ void load_scan(const float* __restrict__ p, int nvalid, float (&out)[V])
{
    if (KEEP && nvalid == 4) {
        const f4 t = *reinterpret_cast<const f4*>(p);
        out[0] = t.x; out[1] = t.y; out[2] = t.z; out[3] = t.w;
    } else {
        load_v<V>(p, nvalid, out);
    }
}

// max |g + e| (g == null: max |e|) over the flat range [start, start + len) wherever it begins: a
// maximum does not care which lane sees which element, so the range is walked as the aligned quads of
// memory it contains plus at most three single elements at either end.  thr != 0: e is read only for
// quads (elements) whose |g| reaches thr (filtered scale pass).
template <bool KEEP>
__device__ __forceinline__ uint32_t amax_range(const float* __restrict__ g, const float* __restrict__ e,
                                               int64_t start, int len, uint32_t thr)
{
    const int64_t end = start + len;
    int64_t a0 = (start + 3) & ~(int64_t)3;
    a0 = a0 < end ? a0 : end;
    int64_t a1 = end & ~(int64_t)3;
    a1 = a1 > a0 ? a1 : a0;
    uint32_t local = 0;
    const int head = (int)(a0 - start), tail = (int)(end - a1);
    if ((int)threadIdx.x < head + tail) {
        const int64_t idx = (int)threadIdx.x < head ? start + threadIdx.x : a1 + ((int)threadIdx.x - head);
        const float gv = g ? g[idx] : 0.0f;
        if (thr == 0u || (f2u(gv) & 0x7fffffffu) >= thr) {
            const uint32_t ab = f2u(gv + e[idx]) & 0x7fffffffu;
            local = ab;
        }
    }
    // four quads per lane per trip, their loads issued together (a tile holds at most 1024 quads)
    for (int64_t q0 = a0 + (int64_t)threadIdx.x * 4; q0 < a1; q0 += kBlockThreads * 16) {
        float gv[4][4], ev[4][4];
        bool live[4], cand[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t q = q0 + (int64_t)k * kBlockThreads * 4;
            live[k] = q < a1;
#pragma unroll
            for (int j = 0; j < 4; ++j) { gv[k][j] = 0.0f; ev[k][j] = 0.0f; }
            if (live[k] && g) load_scan<4, KEEP>(g + q, 4, gv[k]);
            if (live[k] && thr == 0u) load_scan<4, KEEP>(e + q, 4, ev[k]);
        }
        if (thr != 0u) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t top = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t ab = f2u(gv[k][j]) & 0x7fffffffu;
                    top = ab > top ? ab : top;
                }
                cand[k] = live[k] && top >= thr;
                if (cand[k]) load_scan<4, KEEP>(e + q0 + (int64_t)k * kBlockThreads * 4, 4, ev[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (thr == 0u ? live[k] : cand[k]) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t ab = f2u(gv[k][j] + ev[k][j]) & 0x7fffffffu;
                    local = ab > local ? ab : local;
                }
            }
        }
    }
    return local;
}

struct Scale {
    float s, inv;
};

// 1/s must be a normal number with full precision for the error bound of the fast quotient, else 0
__device__ __forceinline__ Scale make_scale(uint32_t max_bits)
{
    Scale r;
    r.s = u2f(max_bits);
    const bool ok = r.s >= 0x1p-100f && r.s <= 0x1p100f;
    r.inv = ok ? 1.0f / r.s : 0.0f;
    return r;
}

// what the residual p - Q_g(p) of a step with this scale can reach (a non-finite scale gives a non-finite
// bound, which switches the next step's filter off); the added 2^-140 covers scales so small that s * level
// itself is rounded
__device__ __forceinline__ float residual_bound(float s, float bound_factor) { return s * bound_factor + 0x1p-140f; }

// Scale of the tile's layer for the worker of table row `row`, from where k_reduce_scales left it.
__device__ __forceinline__ Scale stored_scale(const Fold& F, int row, const Tile& t, const float* scales)
{
    Scale r;
    r.s = scales[t.seg];
    r.inv = F.inv_scales[(size_t)row * F.num_segments + t.seg];
    return r;
}

// Maximum of part[t0 .. t1) over THREADS threads, this one's share: U loads in flight each.
template <int THREADS, int U = 8>
__device__ __forceinline__ uint32_t fold_maxima(const uint32_t* __restrict__ part, int t0, int t1, int thread)
{
    uint32_t local = 0;
    for (int t = t0 + thread; t < t1; t += THREADS * U) {
        uint32_t v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = t + k * THREADS < t1 ? part[t + k * THREADS] : 0u;
#pragma unroll
        for (int k = 0; k < U; ++k) local = v[k] > local ? v[k] : local;
    }
    return local;
}

// The same, folded by one wavefront from the maxima t0 .. t1 of a row.  In two steps, so that loads for several workers can be under
// way together: each lane's share, then the scale; `first`: the wavefront writes it out if its tile `ti` is the layer's first.
struct FoldRange {
    int t0, t1;
};

__device__ __forceinline__ FoldRange fold_range(const Fold& F, const Tile& t)
{
    FoldRange r;
    r.t0 = F.seg_tile_begin ? F.seg_tile_begin[t.seg] * F.per_tile : 0;
    r.t1 = F.seg_tile_begin ? F.seg_tile_begin[t.seg + 1] * F.per_tile : F.row;
    return r;
}

__device__ __forceinline__ uint32_t fold_share(const Fold& F, int row, const FoldRange& r)
{
    const uint32_t* part = F.tile_max + (size_t)row * F.row;
    // Four loads in flight where a lane has several (one after the other / eight / four: one worker's call of 512 tiles
    // 13.5 / 12.3 / 12.4 us, 768 tiles 17.7 / 15.8 / 15.5; step of 4 workers of 16 tiles, one load each, 12.8 / 13.1 / 12.7).
    if (r.t1 - r.t0 > 64) return fold_maxima<64, 4>(part, r.t0, r.t1, (int)threadIdx.x);
    return r.t0 + (int)threadIdx.x < r.t1 ? part[r.t0 + (int)threadIdx.x] : 0u;
}

__device__ __forceinline__ Scale folded_scale(const Fold& F, int row, const Tile& t, int ti, const FoldRange& range, uint32_t share,
                                              bool first, float* scales)
{
    const Scale r = make_scale((uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(share)));
    if (first && ti * F.per_tile == range.t0 && threadIdx.x == 0) {
        scales[t.seg] = r.s;
        F.inv_scales[(size_t)row * F.num_segments + t.seg] = r.inv;
        F.err_bound[(size_t)row * F.num_segments + t.seg] = residual_bound(r.s, F.bound_factor);
    }
    return r;
}

__device__ __forceinline__ Scale folded_scale(const Fold& F, int row, const Tile& t, int ti, bool first, float* scales)
{
    const FoldRange range = fold_range(F, t);
    return folded_scale(F, row, t, ti, range, fold_share(F, row, range), first, scales);
}

__device__ __forceinline__ void check_scale(float s, uint32_t* status)
{
    if (!(s >= 0.0f && s < __builtin_inff()) && threadIdx.x == 0) atomicOr(status, QADAM_STATUS_NONFINITE_SCALE);
}

__device__ __forceinline__ void write_scale(const ScaleArgs& A, int w, int l, uint32_t max_bits)
{
    const Scale r = make_scale(max_bits);
    A.scales[w][l] = r.s;
    A.inv_scales[(size_t)w * A.num_segments + l] = r.inv;
    A.err_bound[(size_t)w * A.num_segments + l] = residual_bound(r.s, A.bound_factor);
}

// grid: (layers, workers).  One workgroup folds the maxima of its (worker, layer).  The maxima come from L2 and
// what bounds the kernel is the chain of loads of one thread, hence 1024 threads and eight loads in flight each.
__global__ void __launch_bounds__(kReduceThreads) k_reduce_scales(ScaleArgs A)
{
    const int l = A.layers ? A.layers[blockIdx.x] : (int)blockIdx.x, w = A.first_worker + blockIdx.y;
    // no table: a single segment that owns every tile
    const int t0 = (A.seg_tile_begin ? A.seg_tile_begin[l] : 0) * A.max_per_tile;
    const int t1 = (A.seg_tile_begin ? A.seg_tile_begin[l + 1] : A.num_tiles) * A.max_per_tile;
    const uint32_t local = fold_maxima<kReduceThreads>(A.tile_max + (size_t)w * A.row, t0, t1, (int)threadIdx.x);
    const uint32_t bm = block_max<kReduceThreads>(local);
    if (threadIdx.x == 0) write_scale(A, w, l, bm);
}

// The same for lists of many layers.  grid: (layers / kListLayers, workers).  Each wavefront folds one layer if its
// maxima are one turn of it (kListMaxima); the longer layers among the workgroup's are folded by all of it afterwards,
// one by one, so that no mix of short and long layers leaves it with one wavefront at work.
__global__ void __launch_bounds__(kReduceThreads) k_reduce_scales_list(ScaleArgs A)
{
    const int first = blockIdx.x * kListLayers, w = A.first_worker + blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t* part = A.tile_max + (size_t)w * A.row;
    // lane k holds layer first + k and its range (past the last layer: an empty one)
    const bool live = lane < kListLayers && first + lane < A.num_layers;
    const int layer = !live ? 0 : A.layers ? A.layers[first + lane] : first + lane;
    const int begin = live ? A.seg_tile_begin[layer] * A.max_per_tile : 0;
    const int end = live ? A.seg_tile_begin[layer + 1] * A.max_per_tile : 0;
    const int t0 = __shfl(begin, wave, 64), t1 = __shfl(end, wave, 64), l = __shfl(layer, wave, 64);
    if (first + wave < A.num_layers && t1 - t0 <= kListMaxima) {
        const uint32_t m = wave_max_u32(fold_maxima<64>(part, t0, t1, lane));
        if (lane == 0) write_scale(A, w, l, m);
    }
#pragma unroll 1
    for (int k = 0; k < kListLayers; ++k) {
        const int a = __builtin_amdgcn_readlane(begin, k), b = __builtin_amdgcn_readlane(end, k);
        if (b - a <= kListMaxima) continue;         // the same in every wavefront of the workgroup
        const uint32_t bm = block_max<kReduceThreads>(fold_maxima<kReduceThreads>(part, a, b, (int)threadIdx.x));
        if (threadIdx.x == 0) write_scale(A, w, __builtin_amdgcn_readlane(layer, k), bm);
        __syncthreads();                            // block_max's parts are read before the next round writes them
    }
}

// Filtered scale pass, stage 2 of 4.  grid: (layers, workers).  The sampled tiles (every
// sample_stride-th of a layer) have their exact maxima: their max is a lower bound LB of the
// layer's scale.  With |e_j| <= B (the bound left by the previous step), an element with
// |g_j| < LB - B has |g_j + e_j| < LB and cannot be the maximum, so the next stage reads e only
// where |g_j| >= thr = (LB - B) minus a safety margin that covers the rounding of g + e.
__global__ void __launch_bounds__(kBlockThreads) k_reduce_lower_bounds(ScaleArgs A)
{
    const int l = A.layers ? A.layers[blockIdx.x] : (int)blockIdx.x, w = A.first_worker + blockIdx.y;
    const int t0 = A.seg_tile_begin[l], t1 = A.seg_tile_begin[l + 1];
    const uint32_t* part = A.tile_max + (size_t)w * A.row;
    uint32_t local = 0;
    for (int t = t0 + (int)threadIdx.x * A.sample_stride; t < t1; t += kBlockThreads * A.sample_stride) {
        const uint32_t v = part[t];
        local = v > local ? v : local;
    }
    const uint32_t bm = block_max(local);
    if (threadIdx.x == 0) {
        const float lb = u2f(bm);
        const float bound = A.err_bound[(size_t)w * A.num_segments + l];
        const float thr = (lb - bound * 1.001f) * 0.999f;
        const bool usable = thr > 0.0f && thr < __builtin_inff() && lb < __builtin_inff();
        A.thr[(size_t)w * A.num_segments + l] = usable ? f2u(thr) : 0u;
    }
}

template <int V, bool KEEP>
__device__ __forceinline__ uint32_t amax_tile(const float* __restrict__ g, const float* __restrict__ e, const Tile& t)
{
    constexpr int BLOCK_ELEMS = kBlockThreads * V;
    uint32_t local = 0;
    if constexpr (V == 4) {
        if (t.len == 4 * BLOCK_ELEMS) {
            // full 4096-element tile: all eight loads of the lane in flight at once
            float gv[4][4], ev[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                load_scan<4, KEEP>(g + t.start + k * BLOCK_ELEMS + threadIdx.x * 4, 4, gv[k]);
                load_scan<4, KEEP>(e + t.start + k * BLOCK_ELEMS + threadIdx.x * 4, 4, ev[k]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t ab = f2u(gv[k][j] + ev[k][j]) & 0x7fffffffu;
                    local = ab > local ? ab : local;
                }
            return local;
        }
    }
    for (int off = threadIdx.x * V; off < t.len; off += BLOCK_ELEMS) {
        const int nvalid = min(t.len - off, V);
        float gv[V], ev[V];
        load_scan<V, KEEP>(g + t.start + off, nvalid, gv);
        load_scan<V, KEEP>(e + t.start + off, nvalid, ev);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const uint32_t ab = f2u(gv[j] + ev[j]) & 0x7fffffffu;
            local = ab > local ? ab : local;
        }
    }
    return local;
}

// grid: (tiles, workers)
template <bool KEEP>
__global__ void __launch_bounds__(kBlockThreads) k_amax(AmaxArgs A)
{
    int ti = (int)blockIdx.x;
    if (KEEP) {
        ti = (int)wave_item(A.items);
        if (ti >= A.num_tiles) return;
    } else if (A.tile_list) {
        ti = A.tile_list[blockIdx.x];
    }
    const Tile t = tile_at(A.tiles, ti, A.seg_len, 0);
    const int w = A.first_worker + blockIdx.y;
    const float* g = A.grad[w];
    const float* e = A.err[w];
    uint32_t local;
    if (t.flags & kTileUnaligned) local = amax_range<KEEP>(g, e, t.start, t.len, 0u);
    else local = amax_tile<4, KEEP>(g, e, t);
    const uint32_t bm = block_max(local);
    if (threadIdx.x == 0) A.tile_max[(size_t)w * A.row + ti] = bm;
}

// Filtered scale pass, stage 3 of 4: max |g + e| over the elements of a tile that can still be the
// layer's maximum, i.e. those with |g| >= thr; e is read for those only.  Comparing bit patterns
// makes a NaN or Inf in g a candidate, so it still surfaces in the scale.
template <int V>
__device__ __forceinline__ uint32_t amax_tile_filtered(const float* __restrict__ g, const float* __restrict__ e,
                                                       const Tile& t, uint32_t thr)
{
    constexpr int BLOCK_ELEMS = kBlockThreads * V;
    uint32_t local = 0;
    if constexpr (V == 4) {
        if (t.len == 4 * BLOCK_ELEMS) {
            float gv[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) load_v<4>(g + t.start + k * BLOCK_ELEMS + threadIdx.x * 4, 4, gv[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                uint32_t top = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t ab = f2u(gv[k][j]) & 0x7fffffffu;
                    top = ab > top ? ab : top;
                }
                if (top >= thr) {
                    float ev[4];
                    load_v<4>(e + t.start + k * BLOCK_ELEMS + threadIdx.x * 4, 4, ev);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t ab = f2u(gv[k][j] + ev[j]) & 0x7fffffffu;
                        local = ab > local ? ab : local;
                    }
                }
            }
            return local;
        }
    }
    for (int off = threadIdx.x * V; off < t.len; off += BLOCK_ELEMS) {
        const int nvalid = min(t.len - off, V);
        float gv[V], ev[V];
        load_v<V>(g + t.start + off, nvalid, gv);
        uint32_t top = 0;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const uint32_t ab = f2u(gv[j]) & 0x7fffffffu;
            top = ab > top ? ab : top;
        }
        if (top >= thr) {
            load_v<V>(e + t.start + off, nvalid, ev);
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const uint32_t ab = f2u(gv[j] + ev[j]) & 0x7fffffffu;
                local = ab > local ? ab : local;
            }
        }
    }
    return local;
}

// grid: (tiles, workers).  Sampled tiles keep the exact maximum stage 1 stored for them.
__global__ void __launch_bounds__(kBlockThreads) k_amax_filtered(AmaxArgs A)
{
    const int ti = blockIdx.x;
    const Tile t = A.tiles[ti];
    if (t.flags & kTileSampled) return;
    const int w = A.first_worker + blockIdx.y;
    const float* g = A.grad[w];
    const float* e = A.err[w];
    const uint32_t thr = A.thr[(size_t)w * A.num_segments + t.seg];
    uint32_t local;
    if (t.flags & kTileUnaligned) local = amax_range<false>(g, e, t.start, t.len, thr);
    else if (thr == 0u) local = amax_tile<4, false>(g, e, t);
    else local = amax_tile_filtered<4>(g, e, t, thr);
    const uint32_t bm = block_max(local);
    if (threadIdx.x == 0) A.tile_max[(size_t)w * A.row + ti] = bm;
}

// max |e| over a tile
template <int V>
__device__ __forceinline__ uint32_t emax_tile(const float* __restrict__ e, const Tile& t)
{
    uint32_t local = 0;
    for (int off = threadIdx.x * V; off < t.len; off += kBlockThreads * V) {
        const int nvalid = min(t.len - off, V);
        float ev[V];
        load_v<V>(e + t.start + off, nvalid, ev);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const uint32_t ab = f2u(ev[j]) & 0x7fffffffu;
            local = ab > local ? ab : local;
        }
    }
    return local;
}

// Verification of the contract behind the filtered pass (bring-up aid): every |e_j| must be within
// the bound the previous step recorded for its layer.  grid: (tiles, workers); reads e only.
__global__ void __launch_bounds__(kBlockThreads) k_check_error_bounds(AmaxArgs A)
{
    const int ti = blockIdx.x;
    const Tile t = A.tiles[ti];
    const int w = A.first_worker + blockIdx.y;
    const float* e = A.err[w];
    const uint32_t local = (t.flags & kTileUnaligned) ? amax_range<false>(nullptr, e, t.start, t.len, 0u) : emax_tile<4>(e, t);
    const uint32_t bm = block_max(local);
    if (threadIdx.x == 0) {
        const float bound = A.err_bound[(size_t)w * A.num_segments + t.seg];
        // a NaN or Inf in e, or a magnitude beyond a finite bound, breaks the contract
        const bool finite_bound = bound < __builtin_inff();
        if (finite_bound && !(u2f(bm) <= bound)) atomicOr(A.status, QADAM_STATUS_ERR_BOUND_VIOLATED);
    }
}

// ------------------------------------------------------------------------------------------------
// common tile walk: every wave of the block takes 64*V elements per iteration; the trip count is
// wave-uniform so the cross-lane packing always runs with all lanes active.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void write_pad_words(uint32_t* codes, const Tile& t, int code_bits)
{
    const int pad = (t.flags >> 8) & 3;
    if ((int)threadIdx.x < pad) {
        const int64_t groups = (t.len + 31) / 32;
        codes[t.code_word + groups * code_bits + threadIdx.x] = 0u;
    }
}

__device__ __forceinline__ void store_chunk_words(uint32_t* __restrict__ codes, const Tile& t, int base,
                                                  int code_bits, uint32_t word, int word_slot, bool writes)
{
    // first element of the group this lane's word belongs to
    const int grp = word_slot / code_bits;
    const bool group_live = base + grp * 32 < t.len;
    if (writes && group_live) {
        const int64_t cw = t.code_word + (int64_t)(base >> 5) * code_bits;
        // an ordinary store: a wavefront's words are 64..128 bytes, less than a line, and L2 puts the pieces of
        // a line together before it goes out (with the non-temporal hint they leave one by one: main pass of
        // 11.7 M parameters, 4 workers, 178 us against 167)
        codes[cw + word_slot] = word;
    }
}

// Two runs of 256 elements per wavefront: one leaves too little in flight behind one wavefront's start-up, four
// start too late (124 M parameters, 4 workers through the separate calls: 2294 / 2246 / 2313 us per step; 2^24
// elements, one worker: 61.3 / 57.5 / 59.9 us).
constexpr int kQuantizeRuns = 2;
constexpr int kQuantizeElems = 256 * kQuantizeRuns;

// ---- worker side alone (qadam_worker_quantize, second pass of variant W) -------------------------
// One turn of a wavefront: C runs of 64 V consecutive elements of a tile from `part_begin`, their loads issued
// together.  FULL: the turn is whole, so that no access needs a guard.
template <int V, int ROUNDING, bool PARKED, bool SH, int C, bool FULL>
__device__ __forceinline__ void worker_part(const WorkerArgs& A, const Tile& t, int ti, int part_begin)
{
    constexpr int WAVE_ELEMS = 64 * V;
    const StepScalars& S = A.S;
    const int lane = threadIdx.x;
    const QgConst c = make_qg(S.k_g);
    const Shift sf = make_shift(t);
    float g[C][V], e[C][V];
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const int off = part_begin + k * WAVE_ELEMS + lane * V;
        const int nvalid = FULL ? V : min(max(t.len - off, 0), V);
        if constexpr (PARKED) {
            // the first pass left p = u + e in the error buffer
            ld<V, SH>(A.err, t.start + off, nvalid, sf, g[k]);
        } else {
            ld<V, SH>(A.grad, t.start + off, nvalid, sf, g[k]);
            ld<V, SH>(A.err, t.start + off, nvalid, sf, e[k]);
        }
    }
    const Scale sc = A.fold.tile_max ? folded_scale(A.fold, 0, t, ti, part_begin == 0, A.scales)
                                     : stored_scale(A.fold, 0, t, A.scales);
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const int base = part_begin + k * WAVE_ELEMS;
        if (!FULL && base >= t.len) break;
        const int off = base + lane * V;
        const int nvalid = FULL ? V : min(max(t.len - off, 0), V);
        const int64_t gi = t.start + off;
        float p[V], unused[V], en[V], U[V];
#pragma unroll
        for (int j = 0; j < V; ++j) { p[j] = PARKED ? g[k][j] : g[k][j] + e[k][j]; unused[j] = 0.0f; U[j] = 0.0f; }
        if constexpr (ROUNDING == 1) unif<V, SH>(S, gi, (uint32_t)A.worker, 0u, sf, U);
        uint32_t codes;
        worker_lane<ROUNDING>(p, sc.s, sc.inv, c, S.mu_bits, U, unused, en, codes);
        st<V, SH>(A.err, gi, nvalid, sf, en);
        int slot; bool writes;
        const uint32_t word = pack_planes(codes, S.code_bits, lane, slot, writes);
        store_chunk_words(A.codes, t, base, S.code_bits, word, slot, writes);
    }
    if (part_begin + C * WAVE_ELEMS >= t.len) write_pad_words(A.codes, t, S.code_bits);
    if (part_begin == 0) check_scale(sc.s, A.status);
}

// LONG: pieces of more than one turn.  The loop over them costs the kernel without it 19 vector registers and 3 to 9 % where
// the launch is short (8 layers of 128 tiles, worker-moments call, 33.0 -> 36.1 us).
template <int ROUNDING, bool PARKED, bool LONG>
__global__ void __launch_bounds__(64) k_worker_quantize(WorkerArgs A)
{
    const uint32_t item = wave_item(A.items);
    if (item >= A.items.count) return;
    const int ti = (int)(item / A.items.cut.parts);
    const Tile t = tile_at(A.tiles, ti, A.seg_len, A.S.code_bits);
    const int part_begin = (int)(item % A.items.cut.parts) * A.items.cut.part_len;
    const int part_end = LONG ? min(t.len, part_begin + A.items.cut.part_len) : t.len;
    int begin = part_begin;
    do {
        if (begin >= part_end) return;
        const bool full = begin + kQuantizeElems <= t.len;
        if (t.flags & kTileUnaligned) {
            if (full) worker_part<4, ROUNDING, PARKED, true, kQuantizeRuns, true>(A, t, ti, begin);
            else worker_part<4, ROUNDING, PARKED, true, kQuantizeRuns, false>(A, t, ti, begin);
        } else {
            if (full) worker_part<4, ROUNDING, PARKED, false, kQuantizeRuns, true>(A, t, ti, begin);
            else worker_part<4, ROUNDING, PARKED, false, kQuantizeRuns, false>(A, t, ti, begin);
        }
        begin += kQuantizeElems;
    } while (LONG);
}

static dim3 wave_grid(const Items& I) { return dim3(wave_blocks(I)); }

template <bool LONG>
static void launch_quantizer(const WorkerArgs& A, hipStream_t stream)
{
    const dim3 grid = wave_grid(A.items), block(64);
    const bool parked = (A.grad == nullptr);
    if (A.S.rounding == 0) {
        if (parked) hipLaunchKernelGGL((k_worker_quantize<0, true, LONG>), grid, block, 0, stream, A);
        else hipLaunchKernelGGL((k_worker_quantize<0, false, LONG>), grid, block, 0, stream, A);
    } else {
        if (parked) hipLaunchKernelGGL((k_worker_quantize<1, true, LONG>), grid, block, 0, stream, A);
        else hipLaunchKernelGGL((k_worker_quantize<1, false, LONG>), grid, block, 0, stream, A);
    }
}

static void launch_quantizer(const WorkerArgs& A, hipStream_t stream)
{
    if (A.items.cut.part_len > kQuantizeElems) launch_quantizer<true>(A, stream);
    else launch_quantizer<false>(A, stream);
}

__device__ __forceinline__ void wait_for_loads()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);         // vmcnt(0)
    asm volatile("" ::: "memory");
}

// ---- a short segment in one workgroup (qadam_quantize_segment_noalloc) ---------------------------
// Scale and quantization in one launch: g and e are read once and p stays in registers across the reduction.
// Bound by latency: one load, two barriers, one store.  10 k elements 13.4 -> 9.5 us per call against the two
// launches of longer segments (16 k: 12.7 -> 9.8); at 32 k one CU's share of the memory is the slower way
// (13.3 -> 13.7).
constexpr int kSegmentThreads = 1024, kSegmentRuns = 4;
constexpr int kSegmentElems = kSegmentThreads * 4 * kSegmentRuns;

struct SegmentArgs {
    StepScalars S;
    const float* grad;
    float* err;
    uint32_t* codes;
    float* scale;
    int n;                     // 1 .. kSegmentElems
};

__global__ void __launch_bounds__(kSegmentThreads) k_segment(SegmentArgs A)
{
    const StepScalars& S = A.S;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const QgConst c = make_qg(S.k_g);
    float p[kSegmentRuns][4];
    uint32_t local = 0;
#pragma unroll
    for (int k = 0; k < kSegmentRuns; ++k) {
        const int off = (k * kSegmentThreads + (int)threadIdx.x) * 4;
        const int nvalid = min(max(A.n - off, 0), 4);
        float g[4], e[4];
        load_v<4>(A.grad + off, nvalid, g);
        load_v<4>(A.err + off, nvalid, e);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            p[k][j] = g[j] + e[j];
            const uint32_t ab = f2u(p[k][j]) & 0x7fffffffu;
            local = ab > local ? ab : local;
        }
    }
    const Scale sc = make_scale((uint32_t)__builtin_amdgcn_readfirstlane((int)block_max<kSegmentThreads>(local)));
    if (threadIdx.x == 0) A.scale[0] = sc.s;
#pragma unroll
    for (int k = 0; k < kSegmentRuns; ++k) {
        const int base = (k * (kSegmentThreads / 64) + wave) * 256;
        if (base >= A.n) break;
        const int off = base + lane * 4;
        const float no_uniforms[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float unused[4] = {0.0f, 0.0f, 0.0f, 0.0f}, en[4];
        uint32_t codes;
        worker_lane<0>(p[k], sc.s, sc.inv, c, S.mu_bits, no_uniforms, unused, en, codes);
        store_v<4>(A.err + off, min(max(A.n - off, 0), 4), en);
        int slot; bool writes;
        const uint32_t word = pack_planes(codes, S.code_bits, lane, slot, writes);
        if (writes && base + slot / S.code_bits * 32 < A.n) A.codes[(base >> 5) * S.code_bits + slot] = word;
    }
    // zero words up to a multiple of 16 bytes
    const int used = (A.n + 31) / 32 * S.code_bits;
    if ((int)threadIdx.x < ((used + 3) & ~3) - used) A.codes[used + threadIdx.x] = 0u;
}

// ---- layers that the chip's registers hold: scale and quantization in one launch -----------------
// The workgroups of a layer keep p = g + e on the chip, meet over the layer's scale and then quantize what they hold, so that
// g and e are read once: 12.4 bytes per element for 20.4 of the two passes.  A workgroup holds two units or three, the oldest one in
// LDS, the younger ones in registers.  Each turn it quantizes the oldest one chunk by chunk while the next unit is loaded and the
// others move up, so that loads and stores mix and a layer's units have a turn or two to meet.  In variant W the local moments are
// updated on the way, 28.4 bytes per element for 36.4.  Bound by memory: 85 M elements, one
// worker 257 -> 194 us with two units, layers of 8 to 17 M elements 261 -> 209 with three; beyond the first and last turns 6.45 TB/s
// with two units and 5.92 with three, whose loads in flight are fewer, in variant W 5.80 and 5.64.
// Layers of one unit each, which do not meet, take the same time.  Measured with guarded stores in every turn (206 us): chunks whose loads
// are in flight together, two units, 2 / 4 / 8: 209 / 206 / 220 us (8 spills); three units, 2 / 4 (4 spills): 211 / 228, where 1024 units
// meet 1706 / 1822; workgroups of 256 / 512 / 1024 threads 205 / 206 / 207; half as many workgroups 253; one unit per workgroup, loaded,
// waited for and stored in turn 229.  The forms with three units and those of variant W have 8 to 52 bytes of scratch per lane; with
// three units one word or up to four are stored there before the first turn and read once in a turn, with two none.  A workgroup's first unit is the one of its own number, the others are drawn from a counter in the order of the layers: all dealt out beforehand
// they end 10 us later, all drawn they begin 4 us later, as 512 draws at once take that long.
// A turn that quantizes a whole unit and loads a whole one runs straight through, without a guard around a store: where paths with and
// without stores join, the wait for the loads becomes one for everything (two units, layers of 144 units 200 / 194).  The maxima of a layer
// are folded with up to 1024 loads under way, 16 to a lane; one after the other they kept its workgroups waiting (three units, step of
// 4 workers, layers of 1024 units 1706 / 1671, 768 units 1351 / 1258).
// Measured and not taken: turns without a barrier, whose first wavefront draws, hands in and asks ahead and tells the others through LDS
// (85 M elements 248); the next unit drawn and the scale asked for at the end of the turn before, the arrival counted during the next
// (768 units 303, as units are put aside that a unit drawn too early keeps waiting).
//
// No workgroup depends on another one being resident.  A workgroup claims its first unit when it starts, and a unit that is claimed
// or drawn is held by a running workgroup, which loads it and hands in its maximum without waiting in between.  A workgroup whose
// polls run out, or whose layer has units that are not held yet, puts its unit aside: it leaves it as it is in memory, goes on,
// and loads it once more when the units have run out.  If a first unit is missing, it claims that one and loads it instead.  So
// every unit of a layer that is waited for comes to be held, and the scale comes.
struct ParkedArgs {
    const ParkedUnit* units;
    const ParkedLayer* layers;
    StepScalars S;
    const float* grad[QADAM_MAX_WORKERS];
    float* err[QADAM_MAX_WORKERS];
    uint32_t* codes[QADAM_MAX_WORKERS];
    float* scales[QADAM_MAX_WORKERS];
    float* mw[QADAM_MAX_WORKERS];   // variant W
    float* vw[QADAM_MAX_WORKERS];
    uint32_t* maxima;       // rows of `row` maxima, one row per worker, one maximum per unit
    uint32_t* meeting;      // [N][meeting_words], zero between launches but for the launches counted
    uint32_t* aside;        // [N][num_units]: of a unit put aside, the one its workgroup put aside before it
    float* inv_scales;      // [N][L]
    float* err_bound;       // [N][L]
    float bound_factor;
    int row, meeting_words, num_segments, first_worker, polls;
    uint32_t num_units, total;      // of one worker, of all
    uint32_t* status;
};

constexpr int kParkedFold = 16;                 // maxima of a layer that a lane of its last workgroup loads together
constexpr uint32_t kNoUnit = 0xffffffffu;
constexpr uint32_t kPublished = 0x80000000u;    // marks a published scale, whose own sign bit is 0
// in place of a scale that did not come (kLastPolls); the status word reports it
constexpr uint32_t kNoScale = kPublished | 0x7fc00000u;

// f(0), f(1), .. f(N - 1) with constants, however long f is (an unrolled loop has a limit)
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

__device__ __forceinline__ uint32_t load_agent(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_agent(uint32_t* p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A table that nothing writes while the kernel runs, through the scalar cache: the index is the same in all lanes.
template <typename T>
__device__ __forceinline__ T load_constant(const T* p)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    typedef const __attribute__((address_space(4))) uint32_t* Words;
    const Words from = (Words)(uint64_t)p;
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = from[i];
    T t;
    __builtin_memcpy(&t, w, sizeof(T));
    return t;
}

// A unit and its layer, the same in all lanes.
struct Place {
    ParkedLayer P;
    int unit, w;
    uint32_t* meeting;
};

__device__ __forceinline__ Place place_of(const ParkedArgs& A, uint32_t item)
{
    const ParkedUnit u = load_constant(A.units + item % A.num_units);
    Place q;
    q.P = load_constant(A.layers + u.layer);
    q.unit = u.unit;
    q.w = A.first_worker + (int)(item / A.num_units);
    q.meeting = A.meeting + (size_t)q.w * A.meeting_words + q.P.meeting;
    return q;
}

// by one wavefront
__device__ __forceinline__ void publish_scale(const ParkedArgs& A, const Place& q, uint32_t max_bits)
{
    const int lane = threadIdx.x & 63;
    if (q.P.num_units > 1 && lane < q.P.copies) {
        // Exchanges, whose answers say that the copies are where the others find them and the last to leave clears them,
        // before this workgroup leaves the meeting.
        const uint32_t before = __hip_atomic_exchange(q.meeting + (1 + lane) * kMeetingLine, max_bits | kPublished,
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" : : "v"(before) : "memory");
    }
    if (lane == 0) {
        const Scale r = make_scale(max_bits);
        A.scales[q.w][q.P.t.seg] = r.s;
        A.inv_scales[(size_t)q.w * A.num_segments + q.P.t.seg] = r.inv;
        A.err_bound[(size_t)q.w * A.num_segments + q.P.t.seg] = residual_bound(r.s, A.bound_factor);
    }
}

// Hands in a unit's maximum; whoever comes last publishes the scale.  By one wavefront.
__device__ __forceinline__ void arrive(const ParkedArgs& A, const Place& q, uint32_t bm)
{
    const int lane = threadIdx.x & 63;
    uint32_t* maxima = A.maxima + (size_t)q.w * A.row + q.P.first_unit;
    uint32_t arrived = 0;
    if (lane == 0) {
        // An exchange, whose answer says that the maximum is where the others find it, before the arrival is counted.
        const uint32_t before = __hip_atomic_exchange(maxima + q.unit, bm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" : : "v"(before) : "memory");
        arrived = __hip_atomic_fetch_add(q.meeting, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    arrived = (uint32_t)__builtin_amdgcn_readfirstlane((int)arrived);
    if ((arrived & kArrivals) != (uint32_t)q.P.num_units - 1u) return;
    uint32_t local = 0;
    // all of them at once: the layer's workgroups wait for this
    for (int i = lane; i < q.P.num_units; i += 64 * kParkedFold) {
        uint32_t v[kParkedFold];
#pragma unroll
        for (int k = 0; k < kParkedFold; ++k) v[k] = load_agent(maxima + min(i + k * 64, q.P.num_units - 1));
#pragma unroll
        for (int k = 0; k < kParkedFold; ++k) local = v[k] > local ? v[k] : local;
    }
    publish_scale(A, q, (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(local)));
}

__device__ __forceinline__ uint32_t poll_scale(const Place& q)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)load_agent(q.meeting + (1 + q.unit % q.P.copies) * kMeetingLine));
}

// The counts of a launch, in the first worker's row: the numbers drawn, the launches before this one and, from kClaims on, for
// every first unit the launch that claimed it last.
__device__ __forceinline__ uint32_t* counts_of(const ParkedArgs& A) { return A.meeting + (size_t)A.first_worker * A.meeting_words; }

// By one thread.
__device__ __forceinline__ bool claim(uint32_t* counts, uint32_t unit, uint32_t launch)
{
    return __hip_atomic_exchange(counts + kClaims + unit, launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != launch;
}

// A first unit from `first` to `last` that nobody holds, or kNoUnit.  By one wavefront.  Every workgroup begins to look at another place,
// so that those which look at the same time claim different units.  Where several launches share the chip, most first units have no
// workgroup yet; looked for from the first one on by all, one of them was claimed at a time and the others loaded units again in
// vain.  us per worker's call, four workers on streams of their own, by all / this way, in two passes: layers of 512 units, two 130 / 69, 55, ten
// 233 / 229, 259; of 768, two 135 / 88, 82; of 1024, two 158 / 119, 106; of 384, four 95 / 80, 104.
__device__ __forceinline__ uint32_t unclaimed(const uint32_t* counts, uint32_t first, uint32_t last, uint32_t launch)
{
    if (first >= (uint32_t)kParkedGroups) return kNoUnit;
    const uint32_t num = min(last, (uint32_t)kParkedGroups - 1u) - first + 1u, parts = (num + 63u) / 64u;
    const uint32_t turn = (blockIdx.x / parts) & 63u;
    uint32_t part = blockIdx.x % parts;
    for (uint32_t i = 0; i < parts; ++i, part = part + 1u < parts ? part + 1u : 0u) {
        const uint32_t u = part * 64u + ((threadIdx.x + turn) & 63u);
        const bool free = u < num && load_agent(counts + kClaims + first + u) != launch;
        const uint64_t any = __builtin_amdgcn_ballot_w64(free);
        if (any) return first + part * 64u + (((uint32_t)__builtin_ctzll(any) + turn) & 63u);
    }
    return kNoUnit;
}

// By one thread.  kNoUnit: they have run out.
__device__ __forceinline__ uint32_t draw_unit(const ParkedArgs& A, uint32_t* counts, uint32_t launch)
{
    const uint32_t unit = kParkedGroups + __hip_atomic_fetch_add(counts, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Every workgroup draws until it draws in vain, once, and has claimed or lost its first unit before: nothing more is drawn or
    // claimed in this launch.
    if (unit == A.total + kParkedGroups - 1u) {
        store_agent(counts, 0u);
        store_agent(counts + 1, launch);
    }
    return unit < A.total ? unit : kNoUnit;
}

// What a turn begins with, and what the first wavefront keeps for it.
struct Turn {
    uint32_t word;          // the scale of the unit to quantize, 0: the unit was put aside
    uint32_t next;          // the unit to load, kNoUnit: none is left
    uint32_t again;         // it was put aside before
    uint32_t launch;        // the number of the launch
    uint32_t kept;          // before the first turn the workgroup's own first unit, kNoUnit: another one has it
    uint32_t out;           // the counter has run out
    uint32_t aside;         // the unit that the workgroup put aside last
};

// To every thread: the scale of `item`, a unit of a layer of several (`met`), and the next unit.
__device__ __forceinline__ void begin_turn(const ParkedArgs& A, const Place& q, uint32_t item, bool met, Turn& turn)
{
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) == 0) {
        uint32_t* counts = counts_of(A);
        uint32_t* links = A.aside + (size_t)A.first_worker * A.num_units;
        const uint32_t launch = (uint32_t)__builtin_amdgcn_readfirstlane((int)turn.launch);
        const bool out = __builtin_amdgcn_readfirstlane((int)turn.out) != 0;
        uint32_t word = 0, missing = kNoUnit;
        if (met) {
            const uint32_t first = item - (uint32_t)q.unit, last = first + (uint32_t)q.P.num_units - 1u;     // of the layer's units
            for (int i = 0; i < (out ? kLastPolls : A.polls); ++i) {
                word = poll_scale(q);
                if (word) break;
                if (i % kPollsUnheld == kPollsUnheld - 1) {
                    missing = unclaimed(counts, first, last, launch);
                    if (missing != kNoUnit || (!out && kParkedGroups + load_agent(counts) <= last)) break;
                }
                __builtin_amdgcn_s_sleep(8);
            }
        }
        if (threadIdx.x == 0) {
            if (met && word == 0) {
                if (out && missing == kNoUnit) {
                    word = kNoScale;
                } else {
                    store_agent(links + item, turn.aside);
                    turn.aside = item;
                }
            }
            // Behind the wait: a unit that is held is loaded without another one, so that its layer can be complete.
            uint32_t next = turn.kept, again = 0;
            if (missing != kNoUnit && claim(counts, missing, launch)) next = missing;
            if (next == kNoUnit && !out) {
                next = draw_unit(A, counts, launch);
                turn.out = next == kNoUnit;
            }
            if (next == kNoUnit && turn.aside != kNoUnit) {
                next = turn.aside;
                turn.aside = load_agent(links + next);
                again = 1;
            }
            turn.word = word; turn.next = next; turn.again = again; turn.kept = kNoUnit;
        }
    }
    __syncthreads();
}

// A layer's part of a buffer of one worker, for accesses with one register of offset per lane beside scalar ones.  A layer that is parked
// takes less than 2^31 bytes.  Stores are not buffer stores: with the offset in a scalar register the compiler knows of no wait between
// one and the next write to its registers, and the first word of lanes 12 to 15 of each row of 16 was stored as that write left it.
typedef __amdgpu_buffer_rsrc_t Buf;
typedef __attribute__((address_space(1))) char* Out;

__device__ __forceinline__ uint64_t uniform_address(const void* p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (uint64_t)hi << 32 | lo;
}

__device__ __forceinline__ Buf buffer_of(const void* p)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)uniform_address(p), 0, -1, 0x00020000);
}

__device__ __forceinline__ Out out_of(void* p) { return (Out)uniform_address(p); }

constexpr int kNonTemporal = 2;

__device__ __forceinline__ void load_buffer(Buf b, uint32_t lane_bytes, int bytes, float (&out)[4])
{
    const u4 t = __builtin_amdgcn_raw_buffer_load_b128(b, (int)lane_bytes, bytes, kNonTemporal);
    out[0] = u2f(t.x); out[1] = u2f(t.y); out[2] = u2f(t.z); out[3] = u2f(t.w);
}

__device__ __forceinline__ void store_out(Out to, uint32_t lane_bytes, int bytes, const float (&in)[4])
{
    const f4 t = {in[0], in[1], in[2], in[3]};
    __builtin_nontemporal_store(t, (__attribute__((address_space(1))) f4_a4*)(to + (uint32_t)bytes + lane_bytes));
}

// Quantizes and stores a wavefront's 256 elements from `base`.  WHOLE: all of them are the layer's, so that no store is guarded and
// the wait for loads issued before is not one for the stores as well.
template <int ROUNDING, bool WHOLE>
__device__ __forceinline__ void parked_chunk(const ParkedArgs& A, const QgConst& c, const Place& q, const Scale& sc, int base, float4 v,
                                             Out err, Out code_words)
{
    const StepScalars& S = A.S;
    const int lane = threadIdx.x & 63;
    const int nvalid = WHOLE ? 4 : min(max(q.P.t.len - base - lane * 4, 0), 4);
    const float old[4] = {v.x, v.y, v.z, v.w};
    float unused[4], en[4], U[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { unused[j] = 0.0f; U[j] = 0.0f; }
    if constexpr (ROUNDING == 1) {
        const int64_t gi = q.P.t.start + base + lane * 4;
        const Shift sf = make_shift(q.P.t);
        StepScalars R = S;
        // the keys of the ten rounds are worked out here and not held in registers over the turns
        asm volatile("" : "+s"(R.key0), "+s"(R.key1));
        if (sf.r) uniforms_shifted<false>(R, gi, (uint32_t)q.w, 0u, sf.r, U);
        else uniforms<4, false>(R, gi, (uint32_t)q.w, 0u, U);
    }
    uint32_t codes;
    worker_lane<ROUNDING>(old, sc.s, sc.inv, c, S.mu_bits, U, unused, en, codes);
    if constexpr (WHOLE) {
        store_out(err, (uint32_t)lane * 16u, base * 4, en);
    } else {
        store_shifted(A.err[q.w] + q.P.t.start + base + lane * 4, nvalid, en);
    }
    int slot; bool writes;
    const uint32_t planes = pack_planes(codes, S.code_bits, lane, slot, writes);
    if constexpr (WHOLE) {
        // lanes with no plane of their own store their group's first word once more
        const uint32_t first = (uint32_t)__builtin_amdgcn_ds_bpermute((lane & 56) * 4, (int)planes);
        *(__attribute__((address_space(1))) uint32_t*)(code_words + (uint32_t)((base >> 5) * S.code_bits * 4) + (uint32_t)(writes ? slot : slot - (lane & 7)) * 4u) =
            writes ? planes : first;
    } else {
        store_chunk_words(A.codes[q.w], q.P.t, base, S.code_bits, planes, slot, writes);
    }
}

// HELD: units in registers.  LOADS: chunks whose loads are in flight together.  W: p is the local update and the error, and the local
// moments take their step; those of a unit put aside have taken it already.
template <int ROUNDING, int HELD, int LOADS, bool W>
__global__ void __launch_bounds__(kParkedThreads, 4) k_parked(ParkedArgs A)
{
    const StepScalars& S = A.S;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int mine = (int)threadIdx.x * 4;
    const QgConst c = make_qg(S.k_g);
    extern __shared__ float4 held[];                    // [kParkedChunks][kParkedThreads]
    float p[HELD][kParkedChunks][4];                    // the younger units, the youngest last; the oldest one is in LDS
    uint32_t item = kNoUnit, younger[HELD];             // the oldest one, the younger ones
    uint32_t word = 0, younger_word[HELD];              // their scales where they are known at once
#pragma unroll
    for (int h = 0; h < HELD; ++h) {
        younger[h] = kNoUnit; younger_word[h] = 0;
#pragma unroll
        for (int k = 0; k < kParkedChunks; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) p[h][k][j] = 0.0f;
    }
    uint32_t next = kNoUnit;
    __shared__ Turn turn;
    if (threadIdx.x == 0) {
        uint32_t* counts = counts_of(A);
        turn.launch = counts[1] + 1u;
        turn.kept = claim(counts, blockIdx.x, turn.launch) ? blockIdx.x : kNoUnit;
        turn.out = 0;
        turn.aside = kNoUnit;
    }
#pragma unroll 1
    for (;;) {
        const Place q = place_of(A, item != kNoUnit ? item : next != kNoUnit ? next : 0u);
        bool met = item != kNoUnit && q.P.num_units > 1;
        begin_turn(A, q, item, met, turn);
        next = (uint32_t)__builtin_amdgcn_readfirstlane((int)turn.next);
        const bool again = __builtin_amdgcn_readfirstlane((int)turn.again) != 0;
        if (met) {
            word = turn.word;
            if (__builtin_amdgcn_readfirstlane((int)word) == 0) {
                item = kNoUnit;
                met = false;
            }
        }
        bool any = item != kNoUnit || next != kNoUnit;
#pragma unroll
        for (int h = 0; h < HELD; ++h) any = any || younger[h] != kNoUnit;
        if (!any) break;
        uint32_t departed = 0;
        if (met && threadIdx.x == 0)
            departed = __hip_atomic_fetch_add(q.meeting, kDeparture, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const Place n = place_of(A, next != kNoUnit ? next : 0u);
        const Scale sc = make_scale((uint32_t)__builtin_amdgcn_readfirstlane((int)(word & ~kPublished)));
        const int q_stride = q.P.num_units * kParkedChunk, q_begin = q.unit * kParkedChunk;
        const int n_stride = n.P.num_units * kParkedChunk, n_begin = n.unit * kParkedChunk;
        const bool q_whole = q_begin + (kParkedChunks - 1) * q_stride + kParkedChunk <= q.P.t.len;
        const bool n_whole = n_begin + (kParkedChunks - 1) * n_stride + kParkedChunk <= n.P.t.len;
        const bool straight = item != kNoUnit && next != kNoUnit && q_whole && n_whole && !(W && again);
        const float* n_grad = A.grad[n.w] + n.P.t.start;
        const float* n_err = A.err[n.w] + n.P.t.start;
        const Buf n_grad_buf = buffer_of(n_grad), n_err_buf = buffer_of(n_err);
        const Out q_err = out_of(A.err[q.w] + q.P.t.start), q_codes = out_of(A.codes[q.w] + q.P.t.code_word);
        float* n_mw = nullptr;
        float* n_vw = nullptr;
        if constexpr (W) { n_mw = A.mw[n.w] + n.P.t.start; n_vw = A.vw[n.w] + n.P.t.start; }
        const Buf n_mw_buf = buffer_of(n_mw), n_vw_buf = buffer_of(n_vw);
        const Out n_mw_out = out_of(n_mw), n_vw_out = out_of(n_vw);
        static_for<kParkedChunks / LOADS>([&](auto part) {
            constexpr int k0 = decltype(part)::value * LOADS;
            float g[LOADS][4], e[LOADS][4], mv[LOADS][4], vv[LOADS][4];
            // the younger units move up, the oldest of them to LDS
            auto move_up = [&](int k) {
                held[k * kParkedThreads + threadIdx.x] = make_float4(p[0][k][0], p[0][k][1], p[0][k][2], p[0][k][3]);
#pragma unroll
                for (int h = 0; h + 1 < HELD; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j) p[h][k][j] = p[h + 1][k][j];
                asm volatile("" : : : "memory");
                __builtin_amdgcn_sched_barrier(0);
            };
            auto keep = [&](int k, int j, float v) {
                p[HELD - 1][k0 + k][j] = v;
                asm volatile("" : "+v"(p[HELD - 1][k0 + k][j]) : : "memory");
            };
            if (straight) {
                const uint32_t at = threadIdx.x * 16u;
#pragma unroll
                for (int k = 0; k < LOADS; ++k) {
                    const int base = n_begin + (k0 + k) * n_stride;
                    load_buffer(n_grad_buf, at, base * 4, g[k]);
                    if constexpr (W) {
                        load_buffer(n_mw_buf, at, base * 4, mv[k]);
                        load_buffer(n_vw_buf, at, base * 4, vv[k]);
                    }
                    load_buffer(n_err_buf, at, base * 4, e[k]);
                }
                asm volatile("" : : : "memory");    // the loads are on their way before the arithmetic
#pragma unroll
                for (int k = k0; k < k0 + LOADS; ++k) {
                    parked_chunk<ROUNDING, true>(A, c, q, sc, q_begin + k * q_stride + wave * 256, held[k * kParkedThreads + threadIdx.x],
                                                 q_err, q_codes);
                    move_up(k);
                }
#pragma unroll
                for (int k = 0; k < LOADS; ++k) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if constexpr (W) keep(k, j, adam_step(S, g[k][j], mv[k][j], vv[k][j]) + e[k][j]);
                        else keep(k, j, g[k][j] + e[k][j]);
                    }
                    if constexpr (W) {
                        const int base = n_begin + (k0 + k) * n_stride;
                        store_out(n_mw_out, at, base * 4, mv[k]);
                        store_out(n_vw_out, at, base * 4, vv[k]);
                    }
                }
                return;
            }
            if (next != kNoUnit) {
#pragma unroll
                for (int k = 0; k < LOADS; ++k) {
                    const int base = n_begin + (k0 + k) * n_stride;
                    const int nvalid = n_whole ? 4 : min(max(n.P.t.len - base - mine, 0), 4);
                    load_any(n_grad + base + mine, nvalid, g[k]);
                    if constexpr (W) {
                        load_any(n_mw + base + mine, nvalid, mv[k]);
                        load_any(n_vw + base + mine, nvalid, vv[k]);
                    }
                    load_any(n_err + base + mine, nvalid, e[k]);
                }
            }
            asm volatile("" : : : "memory");
#pragma unroll
            for (int k = k0; k < k0 + LOADS; ++k) {
                const int base = q_begin + k * q_stride + wave * 256;
                if (item != kNoUnit && (q_whole || base < q.P.t.len))
                    parked_chunk<ROUNDING, false>(A, c, q, sc, base, held[k * kParkedThreads + threadIdx.x], q_err, q_codes);
                move_up(k);
            }
            if (next != kNoUnit) {
#pragma unroll
                for (int k = 0; k < LOADS; ++k) {
                    if constexpr (W) {
                        const int base = n_begin + (k0 + k) * n_stride;
                        const int nvalid = n_whole ? 4 : min(max(n.P.t.len - base - mine, 0), 4);
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float u = again ? adam_quotient(S, mv[k][j], vv[k][j]) : adam_step(S, g[k][j], mv[k][j], vv[k][j]);
                            keep(k, j, j < nvalid ? u + e[k][j] : 0.0f);
                        }
                        if (!again) {
                            store_shifted(n_mw + base + mine, nvalid, mv[k]);
                            store_shifted(n_vw + base + mine, nvalid, vv[k]);
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) keep(k, j, g[k][j] + e[k][j]);
                    }
                }
            }
        });
        if (item != kNoUnit) {
            if (q.unit == 0) write_pad_words(A.codes[q.w], q.P.t, S.code_bits);
            check_scale(sc.s, A.status);
        }
        __syncthreads();                        // the words in LDS are read
        // The last one to leave makes the meeting place ready for the next launch.
        if (met && threadIdx.x == 0 && departed / kDeparture == (uint32_t)q.P.num_units - 1u) {
            store_agent(q.meeting, 0u);
            for (int i = 1; i <= q.P.copies; ++i) store_agent(q.meeting + i * kMeetingLine, 0u);
        }
        if (next != kNoUnit) {
            uint32_t local = 0;
#pragma unroll
            for (int k = 0; k < kParkedChunks; ++k)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t ab = f2u(p[HELD - 1][k][j]) & 0x7fffffffu;
                    local = ab > local ? ab : local;
                }
            const uint32_t bm = block_max<kParkedThreads>(local);
            // not by the wavefront that begins the next turn, whose wait goes on beside this one
            if (wave == kParkedThreads / 64 - 1) {
                if (n.P.num_units == 1) publish_scale(A, n, bm);
                else if (!again) arrive(A, n, bm);
            }
            word = bm;                          // of a layer of one unit
        }
        const uint32_t youngest = word;
        item = younger[0];
        word = younger_word[0];
#pragma unroll
        for (int h = 0; h + 1 < HELD; ++h) { younger[h] = younger[h + 1]; younger_word[h] = younger_word[h + 1]; }
        younger[HELD - 1] = next;
        younger_word[HELD - 1] = youngest;
    }
}

// ---- server side (qadam_server_step, qadam_server_apply_w, the last launch of a step by worker) ---
struct ServerArgs {
    const Tile* tiles;
    Items items;
    StepScalars S;          // k_x < 0: no weight codes
    ServerPtrs sp;
    const uint32_t* codes[QADAM_MAX_WORKERS];
    const float* scales[QADAM_MAX_WORKERS];
};

// Server arithmetic of one lane's elements, from the sum of the workers' messages to the weight codes, and its stores.
// W: the server only subtracts the mean message, m and v are not used.
template <int ROUNDING, int V, bool W, bool SH, bool HALVES = false>
__device__ __forceinline__ void server_lane(const StepScalars& S, const ServerPtrs& sp, const float (&acc)[V], float (&xv)[V],
                                            float (&mv)[V], float (&vv)[V], const float (&wi)[V], int64_t gi, int nvalid,
                                            const Shift& sf)
{
    if constexpr (W) {
#pragma unroll
        for (int j = 0; j < V; ++j) xv[j] = xv[j] - mean_over_workers(S, acc[j]);
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const float u = adam_step(S, mean_over_workers(S, acc[j]), mv[j], vv[j]);
            xv[j] = xv[j] - u;
        }
        st<V, SH>(sp.m, gi, nvalid, sf, mv);
        st<V, SH>(sp.v, gi, nvalid, sf, vv);
    }
    st<V, SH>(sp.x, gi, nvalid, sf, xv);
    if (S.k_x >= 0) {                                    // else Q_x is the identity
        float wo[V];
        int jc[V];
        weight_lane<V, ROUNDING, SH, HALVES>(S, xv, wi, gi, sf, wo, jc);
        if (sp.werr) st<V, SH>(sp.werr, gi, nvalid, sf, wo);
        stw<V, SH>(sp.wcodes, S.wcode_bytes, gi, nvalid, sf, jc);
    }
}

constexpr int kServerElems = 256;

// LDS that a workgroup of the server reserves at least, which holds the pass to 26 wavefronts per CU, or to 20 where the code
// words take no LDS: as in the main pass, more of them only spread the accesses over more DRAM pages.  us, as many as fit / 26
// or 20 / 16 wavefronts: 2^26 elements, one worker 300 / 266 / 264, two 304 / 269 / 265, four 306 / 274 / 272, eight 304 / 286
// / 299, sixteen 373 / 377 / 385; 2^24, eight workers 81.0 / 78.3 / 83.7; 2^22, four 23.0 / 23.0 / 23.4.
// With the weights' residual to read as well 20 or 16 are enough (whole step by worker, 26 or 20 / 20 or 16: 2^26 elements,
// two workers 839 / 824, eight 2103 / 2084; 1.3 G, four 20.15 / 20.04 ms).
constexpr unsigned server_lds(bool held, bool residual)
{
    return held ? (residual ? 10240 : 8192) : (residual ? 8192 : 6144);
}

// One word per lane from memory to LDS, lane n's to dst[n], without a register in between.  wait_for_loads before it is read.
__device__ __forceinline__ void load_to_lds(const uint32_t* src, uint32_t* dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) uint32_t*)src,
                                     (__attribute__((address_space(3))) uint32_t*)dst, 4, 0, 0);
}

__device__ __forceinline__ void wait_for_lds()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);         // lgkmcnt(0)
    asm volatile("" ::: "memory");
}

// One worker's message.  The decoded value of a code has two forms, with the same bits (add_decoded).
template <int MU_BITS, bool FAST>
__device__ __forceinline__ void add_message(const uint32_t (&w)[4], float s, int k_g, float (&acc)[4])
{
    const uint32_t pos = (threadIdx.x & 7) * 4u;
    if constexpr (FAST) {
        add_decoded<MU_BITS>(w, pos, s, make_levels(k_g), acc);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = acc[j] + qg_decode_planes<MU_BITS>(w, pos + (uint32_t)j, s, make_qg(k_g));
    }
}

// One turn of a wavefront: 256 elements of a tile from `base`.  MU_BITS: bits of the level index (code bits minus the sign).
// FULL: the turn is whole, so that no access needs a guard.  U: the number of workers, whose code words and scales are held
// in registers; 0: any number of workers, whose words go through LDS, so that one narrow load per worker brings what the lanes
// of a group share and all workers' loads are under way at once.  Bound by memory.  Loads of every lane's own, four workers (or
// one) at a time, and values decoded bit by bit / this way, us: 2^24 elements, three workers 82.1 / 73.1, five 89.2 / 79.5, eight
// 91.7 / 81.5, sixteen 133 / 92; 2^26, sixteen 452 / 372; 2^28, sixteen 1640 / 1440.  Four workers, whose loads were issued
// together before: 274 / 274 at 2^26.  Through LDS / held: 51 k elements, four workers 3.9 / 3.7; 2^22, three 24.5 / 22.9.
template <int MU_BITS, int U, int ROUNDING, bool W, bool SH, bool FULL>
__device__ __forceinline__ void server_part(const ServerArgs& A, const Tile& t, int base)
{
    constexpr int CODE_BITS = MU_BITS + 1, WORDS = 8 * CODE_BITS;
    const StepScalars& S = A.S;
    const int lane = threadIdx.x;
    const int N = S.num_workers;
    const Shift sf = make_shift(t);
    const int off = base + lane * 4;
    const int nvalid = FULL ? 4 : min(max(t.len - off, 0), 4);
    const int64_t gi = t.start + off, cw = t.code_word + (int64_t)(base >> 5) * CODE_BITS;
    float xv[4], mv[4], vv[4], wi[4], acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { wi[j] = 0.0f; acc[j] = 0.0f; }
    // Everything this turn reads is under way before the first of it is used.
    const float* scales = nullptr;
    if constexpr (U == 0) {
        wait_for_lds();                         // what the turn before read
        scales = A.scales[min(lane, N - 1)];
    }
    ld<4, SH>(A.sp.x, gi, nvalid, sf, xv);
    if constexpr (!W) {
        ld<4, SH>(A.sp.m, gi, nvalid, sf, mv);
        ld<4, SH>(A.sp.v, gi, nvalid, sf, vv);
    }
    if (S.weight_ef && S.k_x >= 0) ld<4, SH>(A.sp.werr, gi, nvalid, sf, wi);
    if constexpr (U == 0) {
        // the scales, worker n's in lane n, and the code words, which go straight to LDS
        extern __shared__ uint32_t words[];     // [N][WORDS]
        const float scale = scales[t.seg];
        // the words behind a tile's last group may lie behind the end of the buffer
        if (lane < WORDS && (FULL || base + lane / CODE_BITS * 32 < t.len)) {
#pragma unroll 4
            for (int i = 0; i < N; ++i) load_to_lds(A.codes[i] + cw + lane, words + i * WORDS);
        }
        wait_for_loads();
        const bool fast = __builtin_amdgcn_ballot_w64(!fast_scale(scale)) == 0;
        auto add_all = [&](auto is_fast) {
            const uint32_t* group = words + (lane >> 3) * CODE_BITS;
            for (int i = 0; i < N; ++i, group += WORDS) {
                uint32_t w[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) w[b] = b < CODE_BITS ? group[b] : 0u;
                const float s = u2f((uint32_t)__builtin_amdgcn_readlane((int)f2u(scale), i));
                add_message<MU_BITS, decltype(is_fast)::value>(w, s, S.k_g, acc);
            }
        };
        if (fast) add_all(std::true_type{});
        else add_all(std::false_type{});
    } else {
        uint32_t w[U][4];
        float s[U];
        bool fast = true;
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int b = 0; b < 4; ++b) w[u][b] = 0u;
            if (FULL || nvalid > 0) load_planes<4, MU_BITS>(A.codes[u] + cw, lane, w[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s[u] = A.scales[u][t.seg];
            fast = fast && fast_scale(s[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (fast) add_message<MU_BITS, true>(w[u], s[u], S.k_g, acc);
            else add_message<MU_BITS, false>(w[u], s[u], S.k_g, acc);
        }
    }
    if (!FULL && nvalid == 0) return;
    server_lane<ROUNDING, 4, W, SH>(S, A.sp, acc, xv, mv, vv, wi, gi, nvalid, sf);
}

// LONG: pieces of more than one turn.
template <int MU_BITS, int U, int ROUNDING, bool W, bool LONG>
__global__ void __launch_bounds__(64) k_server_step(ServerArgs A)
{
    const uint32_t item = wave_item(A.items);
    if (item >= A.items.count) return;
    const Tile t = A.tiles[item / A.items.cut.parts];
    const int part_begin = (int)(item % A.items.cut.parts) * A.items.cut.part_len;
    const int part_end = LONG ? min(t.len, part_begin + A.items.cut.part_len) : t.len;
    int base = part_begin;
    do {
        if (base >= part_end) return;
        const bool full = base + kServerElems <= t.len;
        if (t.flags & kTileUnaligned) {
            if (full) server_part<MU_BITS, U, ROUNDING, W, true, true>(A, t, base);
            else server_part<MU_BITS, U, ROUNDING, W, true, false>(A, t, base);
        } else {
            if (full) server_part<MU_BITS, U, ROUNDING, W, false, true>(A, t, base);
            else server_part<MU_BITS, U, ROUNDING, W, false, false>(A, t, base);
        }
        base += kServerElems;
    } while (LONG);
}

// ---- weight quantizer alone (qadam_weight_quantize) ----------------------------------------------
// Index of a workgroup of a flat launch (flat_grid): one dimension of a grid holds fewer than 2^32 work-items, so a very
// long vector takes several rows.
__device__ __forceinline__ int64_t flat_index() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

struct WeightArgs {
    StepScalars S;
    const float* x;
    float* werr;
    void* wcodes;
    int64_t n;
};

// THREADS * PIECES quads per workgroup, PIECES per lane, in memory order.  Bound by HBM (x, e^x in; e^x, codes out) on long
// vectors, where wavefronts that start and end on their own keep reads and writes mixed: 124 M parameters, 4 workers
// through the separate calls, whole step 2302 us with 256 threads and four quads per lane, 2280 with 64 threads and
// two, 2267 with 64 and one.  Where its data is in the cache the rate at which workgroups start bounds it
// (quantize_in_cache).
template <int ROUNDING, int THREADS, int PIECES>
__global__ void __launch_bounds__(THREADS) k_weight_quantize(WeightArgs A)
{
    const StepScalars& S = A.S;
    const int64_t first = 4 * (flat_index() * (THREADS * PIECES) + threadIdx.x);
    float xv[PIECES][4], wi[PIECES][4];
    int nvalid[PIECES];
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
        const int64_t gi = first + k * THREADS * 4;
        nvalid[k] = (int)max((int64_t)0, min((int64_t)4, A.n - gi));
#pragma unroll
        for (int t = 0; t < 4; ++t) wi[k][t] = 0.0f;
        load_v<4>(A.x + gi, nvalid[k], xv[k]);
        if (S.weight_ef) load_v<4>(A.werr + gi, nvalid[k], wi[k]);
    }
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
        if (nvalid[k] == 0) continue;
        const int64_t gi = first + k * THREADS * 4;
        float wo[4];
        int j[4];
        weight_lane<4, ROUNDING>(S, xv[k], wi[k], gi, Shift{}, wo, j);
        if (A.werr) store_v<4>(A.werr + gi, nvalid[k], wo);
        store_wcodes<4>(A.wcodes, S.wcode_bytes, gi, nvalid[k], j);
    }
}

struct DequantArgs {
    const void* wcodes;
    void* xhat;             // float or __half, per the kernel's template argument
    int64_t n;
    int wcode_bytes;
    float inv_two_kx1;
};

// A workgroup per THREADS * PIECES * E consecutive codes, E per lane and piece (E = 4 for fp32 output, 8 for binary16, so
// that an output store is always 128 bits and a wavefront's is one contiguous 1 KiB run).  Bound by the memory's write side
// on long vectors, by the rate at which workgroups start where the data is in the memory-side cache (decode_shape).
template <bool HALF, int CODE_BYTES, int THREADS, int PIECES>
__global__ void __launch_bounds__(THREADS) k_weight_dequantize(DequantArgs A)
{
    constexpr int E = HALF ? 8 : 4;
    constexpr int WORDS = E * CODE_BYTES / 4;           // code words per lane and piece: 1, 2 or 4
    const int64_t base = E * (flat_index() * (THREADS * PIECES) + threadIdx.x);
    uint32_t w[PIECES][WORDS];
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
        const int64_t i = base + k * THREADS * E;
        const char* src = static_cast<const char*>(A.wcodes) + i * CODE_BYTES;
#pragma unroll
        for (int t = 0; t < WORDS; ++t) w[k][t] = 0u;
        if (i + E <= A.n) {
            if constexpr (WORDS == 1) {
                w[k][0] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(src));
            } else if constexpr (WORDS == 2) {
                const u2 v = __builtin_nontemporal_load(reinterpret_cast<const u2*>(src));
                w[k][0] = v.x; w[k][1] = v.y;
            } else {
                const u4 v = __builtin_nontemporal_load(reinterpret_cast<const u4*>(src));
                w[k][0] = v.x; w[k][1] = v.y; w[k][2] = v.z; w[k][3] = v.w;
            }
        } else {
            // ragged end of the vector: code by code
#pragma unroll
            for (int t = 0; t < E; ++t) {
                if (i + t < A.n) {
                    const uint32_t c = CODE_BYTES == 1 ? (uint32_t)(uint8_t)src[t]
                                                       : (uint32_t)reinterpret_cast<const uint16_t*>(src)[t];
                    w[k][t * CODE_BYTES / 4] |= c << (8 * ((t * CODE_BYTES) & 3));
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < PIECES; ++k) {
        const int64_t i = base + k * THREADS * E;
        const bool full = i + E <= A.n;
        float xh[E];
#pragma unroll
        for (int t = 0; t < E; ++t) {
            const uint32_t c = w[k][t * CODE_BYTES / 4] >> (8 * ((t * CODE_BYTES) & 3));
            const int j = CODE_BYTES == 1 ? (int)(int8_t)c : (int)(int16_t)c;
            xh[t] = (float)j * A.inv_two_kx1;
        }
        if constexpr (HALF) {
            __half* out = static_cast<__half*>(A.xhat) + i;
            if (full) {
                u4 v;
                v.x = (uint32_t)__half_as_ushort(__float2half_rn(xh[0])) | ((uint32_t)__half_as_ushort(__float2half_rn(xh[1])) << 16);
                v.y = (uint32_t)__half_as_ushort(__float2half_rn(xh[2])) | ((uint32_t)__half_as_ushort(__float2half_rn(xh[3])) << 16);
                v.z = (uint32_t)__half_as_ushort(__float2half_rn(xh[4])) | ((uint32_t)__half_as_ushort(__float2half_rn(xh[5])) << 16);
                v.w = (uint32_t)__half_as_ushort(__float2half_rn(xh[6])) | ((uint32_t)__half_as_ushort(__float2half_rn(xh[7])) << 16);
                __builtin_nontemporal_store(v, reinterpret_cast<u4*>(out));
            } else {
#pragma unroll
                for (int t = 0; t < E; ++t) if (i + t < A.n) out[t] = __float2half_rn(xh[t]);
            }
        } else {
            float* out = static_cast<float*>(A.xhat) + i;
            if (full) {
                f4 v;
                v.x = xh[0]; v.y = xh[1]; v.z = xh[2]; v.w = xh[3];
                __builtin_nontemporal_store(v, reinterpret_cast<f4*>(out));
            } else {
#pragma unroll
                for (int t = 0; t < E; ++t) if (i + t < A.n) out[t] = xh[t];
            }
        }
    }
}

// ---- the whole step in one pass (qadam_step_fused) -----------------------------------------------
// One wavefront's share: `part_len` elements of a tile from `part_begin`, 64 V at a time, the workers' g and e
// loaded U workers at a time.  FULL: the share is whole, so that no access needs a guard.
// W = false: variant S (workers' g and e in, server moments).  W = true: second pass of variant W
// (the first pass left p_i = alpha m_i / sqrt(v_i + eps) + e_i in the error buffers; the server
// only subtracts the mean message).
template <int ROUNDING, int V, bool W, bool SH, bool FOLD, int U, bool FULL>
__device__ __forceinline__ void fused_part(const FusedArgs& A, const Tile& t, int ti, int part_begin, int part_len)
{
    constexpr int WAVE_ELEMS = 64 * V;
    const StepScalars& S = A.S;
    const int lane = threadIdx.x;
    const QgConst c = make_qg(S.k_g);
    const int N = S.num_workers;
    const Shift sf = make_shift(t);
    const int part_end = min(t.len, part_begin + part_len);
    FoldRange range;
    if constexpr (FOLD) range = fold_range(A.fold, t);
    for (int base = part_begin; base < part_end; base += WAVE_ELEMS) {
        const int off = base + lane * V;
        const int nvalid = FULL ? V : min(max(t.len - off, 0), V);
        const int64_t gi = t.start + off;
        // server state first: its latency hides behind the workers' arithmetic
        float xv[V], mv[V], vv[V], wi[V];
#pragma unroll
        for (int j = 0; j < V; ++j) wi[j] = 0.0f;
        ld<V, SH>(A.sp.x, gi, nvalid, sf, xv);
        if constexpr (!W) {
            ld<V, SH>(A.sp.m, gi, nvalid, sf, mv);
            ld<V, SH>(A.sp.v, gi, nvalid, sf, vv);
        }
        if (S.weight_ef && S.k_x >= 0) ld<V, SH>(A.sp.werr, gi, nvalid, sf, wi);
        float acc[V];
#pragma unroll
        for (int j = 0; j < V; ++j) acc[j] = 0.0f;
        for (int i0 = 0; i0 < N; i0 += U) {
            float g[U][V], e[U][V];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (U > 1 && i0 + u >= N) break;
                if constexpr (W) {
                    ld<V, SH>(A.err[i0 + u], gi, nvalid, sf, g[u]);       // parked p
                } else {
                    ld<V, SH>(A.grad[i0 + u], gi, nvalid, sf, g[u]);
                    ld<V, SH>(A.err[i0 + u], gi, nvalid, sf, e[u]);
                }
            }
            uint32_t share[U];
            if constexpr (FOLD) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (U > 1 && i0 + u >= N) break;
                    share[u] = fold_share(A.fold, i0 + u, range);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u;
                if (U > 1 && i >= N) break;
                Scale sc;
                if constexpr (FOLD) {
                    sc = folded_scale(A.fold, i, t, ti, range, share[u], base == 0, A.scales[i]);
                    if (base == 0) check_scale(sc.s, A.status);
                } else {
                    sc = stored_scale(A.fold, i, t, A.scales[i]);
                }
                const float s = sc.s, inv_s = sc.inv;
                float p[V], en[V], Ur[V];
#pragma unroll
                for (int j = 0; j < V; ++j) { p[j] = W ? g[u][j] : g[u][j] + e[u][j]; Ur[j] = 0.0f; }
                if constexpr (ROUNDING == 1) unif<V, SH, true>(S, gi, (uint32_t)i, 0u, sf, Ur);
                uint32_t codes;
                worker_lane<ROUNDING>(p, s, inv_s, c, S.mu_bits, Ur, acc, en, codes);
                st<V, SH>(A.err[i], gi, nvalid, sf, en);
                int slot; bool writes;
                const uint32_t word = pack_planes(codes, S.code_bits, lane, slot, writes);
                store_chunk_words(A.codes[i], t, base, S.code_bits, word, slot, writes);
            }
        }
        server_lane<ROUNDING, V, W, SH, true>(S, A.sp, acc, xv, mv, vv, wi, gi, nvalid, sf);
    }
    if (part_begin + part_len >= t.len)
        for (int i = 0; i < N; ++i) write_pad_words(A.codes[i], t, S.code_bits);
    if (!FOLD && part_begin == 0)
        for (int i = 0; i < N; ++i) check_scale(A.scales[i][t.seg], A.status);
}

// U: workers whose loads are in flight together.  4: the scales are there.  Else the pass folds them itself, for all U workers' layers at
// once, in whole pieces and in the ends of layers: few wavefronts, each a chain of loads, so that what is under way together decides.
// Beyond about 256 tiles, which few workers alone reach, the registers of five cost more.  us per step, one after the other / two / five
// together: ragged lists of 51 k elements, 4 workers 15.1 / 14.8 / 14.6, 8 21.1 / 19.3 / 19.1, 16 33.7 / 29.8 / 28.4; one layer of 16 tiles, 2
// workers 10.9 / 10.7 / 10.9, 4 12.7 / 12.2 / 12.1, 8 16.8 / 15.5 / 15.2, 16 26.2 / 22.4 / 21.5; of 128, 3 13.0 / 13.1 / 13.0, 5 15.7 / 15.6 /
// 15.4; of 256, 2 16.3 / 16.8 / 19.8, 4 22.4 / 20.3 / 25.1; variant W, ragged, 8 workers 20.8 / 18.8 / 18.3.
constexpr int kFoldFew = 2, kFoldMany = 5;

template <int ROUNDING, int U, bool W>
__global__ void __launch_bounds__(64) k_fused(FusedArgs A)
{
    constexpr bool FOLD = U != 4;
    const uint32_t item = wave_item(A.items);
    if (item >= A.items.count) return;
    const int ti = (int)(item / A.items.cut.parts);
    const Tile t = A.tiles[ti];
    const int part_len = A.items.cut.part_len;
    const int part_begin = (int)(item % A.items.cut.parts) * part_len;
    if (part_begin >= t.len) return;
    const bool full = part_begin + part_len <= t.len;
    if (t.flags & kTileUnaligned) {
        if (full) fused_part<ROUNDING, 4, W, true, FOLD, U, true>(A, t, ti, part_begin, part_len);
        else fused_part<ROUNDING, 4, W, true, FOLD, FOLD ? U : 1, false>(A, t, ti, part_begin, part_len);
    } else {
        if (full) fused_part<ROUNDING, 4, W, false, FOLD, U, true>(A, t, ti, part_begin, part_len);
        else fused_part<ROUNDING, 4, W, false, FOLD, FOLD ? U : 1, false>(A, t, ti, part_begin, part_len);
    }
}

// ---- short layers: scale and quantization in one go ----------------------------------------------
struct LayerArgs {
    const Tile* tiles;              // a tile for each layer
    Items items;
    uint32_t* status;
    StepScalars S;
    ServerPtrs sp;                  // SERVER only
    const float* grad[QADAM_MAX_WORKERS];
    float* mw[QADAM_MAX_WORKERS];   // variant W only
    float* vw[QADAM_MAX_WORKERS];
    float* err[QADAM_MAX_WORKERS];
    uint32_t* codes[QADAM_MAX_WORKERS];
    float* scales[QADAM_MAX_WORKERS];
    float* err_bound;               // [N][L]
    float bound_factor;
    int first_worker, num_segments;
};

// A layer of THREADS * C * 4 elements or fewer: p of one worker stays in registers between the scale and the quantizer, the
// sum of the messages until the server's part, so everything is read once.  SERVER: the whole step of all workers, else one
// worker's call.  Bound by memory where there are thousands of layers (20000 of 1000 elements, 4 workers: 1.65 GB in 298
// us), by one worker's chain after the other's where there are few.  One quad per lane wherever the layer fits: with one
// wavefront and four quads 20000 layers of 997 took 362 us for 335, and 300 of 1000 22.9 for 12.6.
template <int ROUNDING, int THREADS, int C, bool SERVER, bool W, bool SH>
__device__ __forceinline__ void layer_step(const LayerArgs& A, const Tile& t)
{
    const StepScalars& S = A.S;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const QgConst c = make_qg(S.k_g);
    const Shift sf = make_shift(t);
    const int num = SERVER ? S.num_workers : 1;
    // The next worker's loads, behind the last one's the server's, are under way while this one's maximum is found, where that
    // leaves enough wavefronts per SIMD (us per step of 4 workers, without / with the next worker's: 20000 layers of 997
    // elements 362 / 335, 10000 of 2000 296 / 346; with the next worker's / the server's too, 20000 of 1000: 299 / 289, one
    // worker 160 / 158).
    constexpr bool AHEAD = C == 1;
    int base[C], nvalid[C];
    int64_t gi[C];
    float acc[C][4];
#pragma unroll
    for (int k = 0; k < C; ++k) {
        base[k] = (k * (THREADS / 64) + wave) * 256;
        const int off = base[k] + lane * 4;
        nvalid[k] = min(max(t.len - off, 0), 4);
        gi[k] = t.start + off;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[k][j] = 0.0f;
    }
    // what worker i brings; W: the local moments too
    float g[C][4], e[C][4], lm[C][4], lv[C][4];
    auto load_worker = [&](int i) {
#pragma unroll
        for (int k = 0; k < C; ++k) {
            ld<4, SH>(A.grad[i], gi[k], nvalid[k], sf, g[k]);
            ld<4, SH>(A.err[i], gi[k], nvalid[k], sf, e[k]);
            if constexpr (W) {
                ld<4, SH>(A.mw[i], gi[k], nvalid[k], sf, lm[k]);
                ld<4, SH>(A.vw[i], gi[k], nvalid[k], sf, lv[k]);
            }
        }
    };
    float x[C][4], m[C][4], v[C][4], wi[C][4];
    auto load_server = [&]() {
#pragma unroll
        for (int k = 0; k < C; ++k) {
#pragma unroll
            for (int j = 0; j < 4; ++j) wi[k][j] = 0.0f;
            ld<4, SH>(A.sp.x, gi[k], nvalid[k], sf, x[k]);
            if constexpr (!W) {
                ld<4, SH>(A.sp.m, gi[k], nvalid[k], sf, m[k]);
                ld<4, SH>(A.sp.v, gi[k], nvalid[k], sf, v[k]);
            }
            if (S.weight_ef && S.k_x >= 0) ld<4, SH>(A.sp.werr, gi[k], nvalid[k], sf, wi[k]);
        }
    };
    if constexpr (AHEAD) load_worker(A.first_worker);
    for (int i = A.first_worker; i < A.first_worker + num; ++i) {
        if constexpr (!AHEAD) load_worker(i);
        float p[C][4];
        uint32_t local = 0;
#pragma unroll
        for (int k = 0; k < C; ++k) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (W) p[k][j] = adam_step(S, g[k][j], lm[k][j], lv[k][j]) + e[k][j];
                else p[k][j] = g[k][j] + e[k][j];
                // beyond the end the step alpha m / sqrt(v + eps) is 0 / 0 where eps is 0; codes there are zero bits
                if (W && j >= nvalid[k]) p[k][j] = 0.0f;
                const uint32_t ab = f2u(p[k][j]) & 0x7fffffffu;
                local = ab > local ? ab : local;
            }
            if constexpr (W) {
                st<4, SH>(A.mw[i], gi[k], nvalid[k], sf, lm[k]);
                st<4, SH>(A.vw[i], gi[k], nvalid[k], sf, lv[k]);
            }
        }
        if (SERVER && AHEAD) {
            if (i + 1 < num) load_worker(i + 1);
            else load_server();
        }
        uint32_t bits = wave_max_u32(local);
        if constexpr (THREADS > 64) {
            // two sets of parts in turn: whoever writes a set for worker i + 2 has passed the barrier of worker i + 1, behind
            // which nobody reads worker i's
            __shared__ uint32_t wave_part[2][THREADS / 64];
            if (lane == 0) wave_part[i & 1][wave] = bits;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < THREADS / 64; ++w) bits = wave_part[i & 1][w] > bits ? wave_part[i & 1][w] : bits;
        }
        const Scale sc = make_scale((uint32_t)__builtin_amdgcn_readfirstlane((int)bits));
        if (threadIdx.x == 0) {
            A.scales[i][t.seg] = sc.s;
            A.err_bound[(size_t)i * A.num_segments + t.seg] = residual_bound(sc.s, A.bound_factor);
        }
        check_scale(sc.s, A.status);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            if (base[k] >= t.len) break;
            float en[4], U[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) U[j] = 0.0f;
            if constexpr (ROUNDING == 1) unif<4, SH>(S, gi[k], (uint32_t)i, 0u, sf, U);
            uint32_t codes;
            worker_lane<ROUNDING>(p[k], sc.s, sc.inv, c, S.mu_bits, U, acc[k], en, codes);
            st<4, SH>(A.err[i], gi[k], nvalid[k], sf, en);
            int slot; bool writes;
            const uint32_t word = pack_planes(codes, S.code_bits, lane, slot, writes);
            store_chunk_words(A.codes[i], t, base[k], S.code_bits, word, slot, writes);
        }
        write_pad_words(A.codes[i], t, S.code_bits);
    }
    if constexpr (SERVER) {
        if constexpr (!AHEAD) load_server();
#pragma unroll
        for (int k = 0; k < C; ++k) {
            if (base[k] >= t.len) break;
            server_lane<ROUNDING, 4, W, SH>(S, A.sp, acc[k], x[k], m[k], v[k], wi[k], gi[k], nvalid[k], sf);
        }
    }
}

template <int ROUNDING, int THREADS, int C, bool SERVER, bool W>
__global__ void __launch_bounds__(THREADS) k_layers(LayerArgs A)
{
    const uint32_t item = wave_item(A.items);
    if (item >= A.items.count) return;
    const Tile t = A.tiles[item];
    if (t.flags & kTileUnaligned) layer_step<ROUNDING, THREADS, C, SERVER, W, true>(A, t);
    else layer_step<ROUNDING, THREADS, C, SERVER, W, false>(A, t);
}

// ---- Q_g = identity: the messages are fp32 values ------------------------------------------------
// W = false: the message of worker i is its gradient (plain distributed generic Adam on the mean
// gradient, then Q_x).  W = true: second pass of variant W with the identity quantizer: the message
// is the parked p_i = alpha m_i / sqrt(v_i + eps) + e_i, all of it is sent, so e_i <- 0.
template <int V, int ROUNDING, int U, bool W, bool SH = false>
__device__ __forceinline__ void plain_tile(const FusedArgs& A, const Tile& t)
{
    constexpr int WAVE_ELEMS = 64 * V, BLOCK_ELEMS = (kBlockThreads / 64) * WAVE_ELEMS;
    const StepScalars& S = A.S;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int N = S.num_workers;
    const bool quantize_x = S.k_x >= 0;
    const Shift sf = make_shift(t);
    for (int base = wave * WAVE_ELEMS; base < t.len; base += BLOCK_ELEMS) {
        const int off = base + lane * V;
        const int nvalid = min(max(t.len - off, 0), V);
        if (nvalid == 0) continue;
        const int64_t gi = t.start + off;
        float xv[V], mv[V], vv[V], wi[V], wo[V], acc[V], zero[V];
        int jc[V];
#pragma unroll
        for (int j = 0; j < V; ++j) { wi[j] = 0.0f; acc[j] = 0.0f; zero[j] = 0.0f; }
        ld<V, SH>(A.sp.x, gi, nvalid, sf, xv);
        if constexpr (!W) {
            ld<V, SH>(A.sp.m, gi, nvalid, sf, mv);
            ld<V, SH>(A.sp.v, gi, nvalid, sf, vv);
        }
        if (S.weight_ef && quantize_x) ld<V, SH>(A.sp.werr, gi, nvalid, sf, wi);
        for (int i0 = 0; i0 < N; i0 += U) {
            float p[U][V];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (W) ld<V, SH>(A.err[i0 + u], gi, nvalid, sf, p[u]);
                else ld<V, SH>(A.grad[i0 + u], gi, nvalid, sf, p[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int j = 0; j < V; ++j) acc[j] = acc[j] + p[u][j];
                if constexpr (W) st<V, SH>(A.err[i0 + u], gi, nvalid, sf, zero);
            }
        }
        if constexpr (W) {
#pragma unroll
            for (int j = 0; j < V; ++j) xv[j] = xv[j] - mean_over_workers(S, acc[j]);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const float u = adam_step(S, mean_over_workers(S, acc[j]), mv[j], vv[j]);
                xv[j] = xv[j] - u;
            }
            st<V, SH>(A.sp.m, gi, nvalid, sf, mv);
            st<V, SH>(A.sp.v, gi, nvalid, sf, vv);
        }
        st<V, SH>(A.sp.x, gi, nvalid, sf, xv);
        if (quantize_x) {
            weight_lane<V, ROUNDING, SH>(S, xv, wi, gi, sf, wo, jc);
            if (A.sp.werr) st<V, SH>(A.sp.werr, gi, nvalid, sf, wo);
            stw<V, SH>(A.sp.wcodes, S.wcode_bytes, gi, nvalid, sf, jc);
        }
    }
}

template <int ROUNDING, int U, bool W>
__global__ void __launch_bounds__(kBlockThreads) k_plain_messages(FusedArgs A)
{
    const int ti = blockIdx.x;
    const Tile t = A.tiles[ti];
    if (t.flags & kTileUnaligned) plain_tile<4, ROUNDING, U, W, true>(A, t);
    else plain_tile<4, ROUNDING, U, W, false>(A, t);
}

// ---- variant W, first pass: local moments, park p = u + e in the error buffer, scale ------------
struct MomentsWArgs {
    const Tile* tiles;
    int row;                // maxima from one worker's to the next's
    StepScalars S;
    const float* grad[QADAM_MAX_WORKERS];
    float* mw[QADAM_MAX_WORKERS];
    float* vw[QADAM_MAX_WORKERS];
    float* err[QADAM_MAX_WORKERS];
    uint32_t* tile_max;     // rows of `row` maxima, cut.parts to a tile
    Cut cut;
    int first_worker;
};

// an ordinary store: the lines stay in the cache in front of the memory for the next pass
template <bool SH>
__device__ __forceinline__ void store_keep(float* __restrict__ p, int nvalid, const float (&in)[4])
{
    if (nvalid == 4) {
        f4 t;
        t.x = in[0]; t.y = in[1]; t.z = in[2]; t.w = in[3];
        if constexpr (SH) *reinterpret_cast<f4_a4*>(p) = t;
        else *reinterpret_cast<f4*>(p) = t;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) if (j < nvalid) p[j] = in[j];
    }
}

template <int V, bool SH, bool KEEP>
__device__ __forceinline__ uint32_t moments_w_part(const StepScalars& S, const float* __restrict__ grad,
                                                   float* __restrict__ mw, float* __restrict__ vw,
                                                   float* __restrict__ err, const Tile& t, int part_begin, int part_len)
{
    constexpr int BLOCK_ELEMS = kBlockThreads * V;
    uint32_t local = 0;
    const Shift sf = make_shift(t);
    for (int base = part_begin; base < min(t.len, part_begin + part_len); base += BLOCK_ELEMS) {
        const int off = base + threadIdx.x * V;
        const int nvalid = min(max(t.len - off, 0), V);
        const int64_t gi = t.start + off;
        float g[V], mv[V], vv[V], e[V], p[V];
        ld<V, SH>(grad, gi, nvalid, sf, g);
        ld<V, SH>(mw, gi, nvalid, sf, mv);
        ld<V, SH>(vw, gi, nvalid, sf, vv);
        ld<V, SH>(err, gi, nvalid, sf, e);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const float u = adam_step(S, g[j], mv[j], vv[j]);
            p[j] = u + e[j];
            const uint32_t ab = j < nvalid ? (f2u(p[j]) & 0x7fffffffu) : 0u;
            local = ab > local ? ab : local;
        }
        st<V, SH>(mw, gi, nvalid, sf, mv);
        st<V, SH>(vw, gi, nvalid, sf, vv);
        if constexpr (KEEP) store_keep<SH>(err + gi, nvalid, p);
        else st<V, SH>(err, gi, nvalid, sf, p);
    }
    return local;
}

// grid: (tiles * cut.parts, workers), one 1024-element turn per workgroup: a workgroup that does a whole tile turn by
// turn leaves the memory idle between a turn's stores and the next one's loads (11.7 M parameters, 4 workers:
// 240 us with whole tiles, 226 with quarters).
template <bool KEEP>
__global__ void __launch_bounds__(kBlockThreads) k_moments_w(MomentsWArgs A)
{
    const int ti = (int)(blockIdx.x / A.cut.parts);
    const Tile t = A.tiles[ti];
    const int part_len = A.cut.part_len, part_begin = (int)(blockIdx.x % A.cut.parts) * part_len;
    const int w = A.first_worker + blockIdx.y;
    uint32_t local;
    if (t.flags & kTileUnaligned)
        local = moments_w_part<4, true, KEEP>(A.S, A.grad[w], A.mw[w], A.vw[w], A.err[w], t, part_begin, part_len);
    else
        local = moments_w_part<4, false, KEEP>(A.S, A.grad[w], A.mw[w], A.vw[w], A.err[w], t, part_begin, part_len);
    const uint32_t bm = block_max(local);
    if (threadIdx.x == 0) A.tile_max[(size_t)w * A.row + blockIdx.x] = bm;
}

// ---- diagnostic: per-layer sum of squares in fp64, fixed order ---------------------------------
struct SumsqArgs {
    const Tile* tiles;
    const float* a;
    const float* b;         // may be null
    double* tile_sum;       // [num_tiles]
    const int32_t* seg_tile_begin;
    double* out;            // [num_segments]
};

// block-wide sum in a fixed order: butterfly inside each wavefront, then the wavefronts in index
// order; every thread gets the result
__device__ __forceinline__ double block_sum_f64(double v)
{
    __shared__ double wave_part[kBlockThreads / 64];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();                       // the array may still be read from an earlier call
    if (lane == 0) wave_part[wave] = v;
    __syncthreads();
    double s = wave_part[0];
#pragma unroll
    for (int w = 1; w < kBlockThreads / 64; ++w) s += wave_part[w];
    return s;
}

template <int V>
__device__ __forceinline__ double sumsq_tile(const float* __restrict__ a, const float* __restrict__ b, const Tile& t)
{
    constexpr int BLOCK_ELEMS = kBlockThreads * V;
    double local = 0.0;
    for (int off = threadIdx.x * V; off < t.len; off += BLOCK_ELEMS) {
        const int nvalid = min(t.len - off, V);
        float av[V], bv[V];
        load_v<V>(a + t.start + off, nvalid, av);
        if (b) {
            load_v<V>(b + t.start + off, nvalid, bv);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) bv[j] = 0.0f;
        }
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const double p = (double)(av[j] + bv[j]);     // the sum in fp32, as the step forms it
            local += p * p;                               // exact product of two 24-bit significands
        }
    }
    return local;
}

// grid: tiles
__global__ void __launch_bounds__(kBlockThreads) k_sumsq_tiles(SumsqArgs A)
{
    const int ti = blockIdx.x;
    const Tile t = A.tiles[ti];
    double local;
    if (t.flags & kTileUnaligned) local = sumsq_tile<1>(A.a, A.b, t);
    else local = sumsq_tile<4>(A.a, A.b, t);
    const double s = block_sum_f64(local);
    if (threadIdx.x == 0) A.tile_sum[ti] = s;
}

// grid: layers.  Thread k adds tiles k, k+256, ... of its layer in that order, then the block sum.
__global__ void __launch_bounds__(kBlockThreads) k_sumsq_layers(SumsqArgs A)
{
    const int l = blockIdx.x;
    const int t0 = A.seg_tile_begin[l], t1 = A.seg_tile_begin[l + 1];
    double local = 0.0;
    for (int t = t0 + threadIdx.x; t < t1; t += kBlockThreads) local += A.tile_sum[t];
    const double s = block_sum_f64(local);
    if (threadIdx.x == 0) A.out[l] = s;
}

}  // namespace

// ================================================================================================
// launchers
// ================================================================================================
// |p - Q_g(p)| <= factor * s: half the widest gap of the grid for nearest rounding (the gap between
// 1/2 and 1, or between 0 and 1 for the ternary grid), the whole gap for stochastic rounding; the
// small excess covers the rounding of the quotient p / s that takes the decision.
static float residual_bound_factor(const StepScalars& S)
{
    const float half_gap = S.k_g >= 1 ? 0.25f : 0.5f;
    return (S.rounding == 0 ? half_gap : 2.0f * half_gap) * (1.0f + 0x1p-20f);
}

static void fill_scale_args(ScaleArgs& A, const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker)
{
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) A.scales[i] = W.scales[i];
    A.inv_scales = L.inv_scales; A.tile_max = L.tile_max; A.row = L.max_row; A.seg_tile_begin = L.scaled.seg_tile_begin;
    A.first_worker = first_worker; A.num_segments = L.num_segments; A.num_tiles = L.scaled.shape.num_tiles;
    A.layers = L.scaled.layers; A.num_layers = L.scaled.num_layers;
    A.err_bound = L.err_bound; A.thr = L.thr;
    A.bound_factor = residual_bound_factor(S);
    A.sample_stride = kSampleStride;
}

static bool fold_in_quantizer(const Launch& L, int num, int max_per_tile)
{
    return !L.parked_done && !L.empty_layers && !L.short_layers
        && fold_in_quantizer(L.num_tiles, L.num_params, L.longest_layer * max_per_tile, num, max_per_tile);
}

static Fold make_fold(const Launch& L, const StepScalars& S, int worker, int num, int max_per_tile)
{
    Fold F;
    F.row = L.max_row; F.per_tile = max_per_tile;
    F.tile_max = fold_in_quantizer(L, num, max_per_tile) ? L.tile_max + (size_t)worker * F.row : nullptr;
    F.seg_tile_begin = L.scaled.seg_tile_begin;
    F.num_segments = L.num_segments;
    F.inv_scales = L.inv_scales + (size_t)worker * L.num_segments;
    F.err_bound = L.err_bound + (size_t)worker * L.num_segments;
    F.bound_factor = residual_bound_factor(S);
    return F;
}

hipError_t launch_reduce_scales(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num,
                                int max_per_tile)
{
    if (L.scaled.num_layers == 0 || num == 0 || fold_in_quantizer(L, num, max_per_tile)) return hipSuccess;
    ScaleArgs A;
    fill_scale_args(A, L, S, W, first_worker);
    A.max_per_tile = max_per_tile;
    const dim3 grid(reduce_blocks(A.num_layers, num), num), block(kReduceThreads);
    if (reduce_by_list(A.num_layers, num)) hipLaunchKernelGGL(k_reduce_scales_list, grid, block, 0, L.stream, A);
    else hipLaunchKernelGGL(k_reduce_scales, grid, block, 0, L.stream, A);
    return hipGetLastError();
}

static void fill_amax_args(AmaxArgs& A, const Launch& L, const WorkerPtrs& W, int first_worker)
{
    A.tiles = L.scaled.tiles; A.num_tiles = L.scaled.shape.num_tiles;
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) { A.grad[i] = W.grad[i]; A.err[i] = W.err[i]; }
    A.tile_max = L.tile_max; A.row = L.max_row;
    A.first_worker = first_worker;
    A.tile_list = nullptr; A.thr = L.thr; A.num_segments = L.num_segments;
    A.err_bound = L.err_bound; A.status = L.status;
    A.seg_len = 0;
}

hipError_t launch_check_error_bounds(const Launch& L, const WorkerPtrs& W, int first_worker, int num)
{
    if (L.num_tiles == 0 || num == 0) return hipSuccess;
    AmaxArgs A;
    fill_amax_args(A, L, W, first_worker);
    A.tiles = L.tiles;      // every layer's
    hipLaunchKernelGGL(k_check_error_bounds, dim3(L.num_tiles, num), dim3(kBlockThreads), 0, L.stream, A);
    return hipGetLastError();
}

static void launch_scan(AmaxArgs& A, const ListShape& shape, int64_t n, int num, hipStream_t stream)
{
    A.items = scan_items(shape);
    if (keep_scanned(n, num) && scan_fits(A.items)) {
        hipLaunchKernelGGL(k_amax<true>, dim3(wave_blocks(A.items), num), dim3(kBlockThreads), 0, stream, A);
    } else {
        hipLaunchKernelGGL(k_amax<false>, dim3(A.num_tiles, num), dim3(kBlockThreads), 0, stream, A);
    }
}

hipError_t launch_amax(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num)
{
    (void)S;
    if (L.scaled.shape.num_tiles == 0 || num == 0) return hipSuccess;
    AmaxArgs A;
    fill_amax_args(A, L, W, first_worker);
    launch_scan(A, L.scaled.shape, L.scaled.num_elems, num, L.stream);
    return hipGetLastError();
}

// The scale pass when every |e_j| is known to be at most the bound the previous step left:
// exact maxima of the sampled tiles -> per-layer thresholds -> the other tiles, reading e only
// where |g| reaches the threshold.  launch_reduce_scales follows as usual.
hipError_t launch_amax_filtered(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num)
{
    if (L.scaled.shape.num_tiles == 0 || num == 0) return hipSuccess;
    AmaxArgs A;
    fill_amax_args(A, L, W, first_worker);
    A.tile_list = L.sample_tiles;
    hipLaunchKernelGGL(k_amax<false>, dim3(L.num_sample_tiles, num), dim3(kBlockThreads), 0, L.stream, A);
    ScaleArgs R;
    fill_scale_args(R, L, S, W, first_worker);
    hipLaunchKernelGGL(k_reduce_lower_bounds, dim3(L.scaled.num_layers, num), dim3(kBlockThreads), 0, L.stream, R);
    A.tile_list = nullptr;
    hipLaunchKernelGGL(k_amax_filtered, dim3(L.scaled.shape.num_tiles, num), dim3(kBlockThreads), 0, L.stream, A);
    return hipGetLastError();
}

static bool codes_overlap(const Launch& L, const WorkerPtrs& W, int first_worker, int num)
{
    for (int i = first_worker + 1; i < first_worker + num; ++i)
        for (int k = first_worker; k < i; ++k)
            if (W.codes[i] < W.codes[k] + L.code_words && W.codes[k] < W.codes[i] + L.code_words) return true;
    return false;
}

// Two code buffers that overlap are left to the main pass, which gives them an order.
bool use_parked(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num, bool call, bool variant_w)
{
    const Parked& P = L.parked;
    const bool worth = variant_w ? worth_parking_w(P.num_elems, P.num_units, L.scaled.num_elems, num, S.rounding == 1, P.longest)
                                 : worth_parking(P.num_elems, P.num_units, L.scaled.num_elems, num, S.rounding == 1, call, P.longest);
    return P.num_units > 0 && worth && !codes_overlap(L, W, first_worker, num);
}

template <int ROUNDING, int HELD, int LOADS, bool W>
static void launch_parked(const ParkedArgs& A, hipStream_t stream)
{
    const unsigned lds = kParkedThreads * kParkedChunks * sizeof(float4);
    hipLaunchKernelGGL((k_parked<ROUNDING, HELD, LOADS, W>), dim3(kParkedGroups), dim3(kParkedThreads), lds, stream, A);
}

template <int ROUNDING>
static void launch_parked(const ParkedArgs& A, bool three, bool variant_w, hipStream_t stream)
{
    if (variant_w) {
        if (three) launch_parked<ROUNDING, 2, 1, true>(A, stream);
        else launch_parked<ROUNDING, 1, 2, true>(A, stream);
    } else {
        if (three) launch_parked<ROUNDING, 2, 2, false>(A, stream);
        else launch_parked<ROUNDING, 1, 4, false>(A, stream);
    }
}

hipError_t launch_parked(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num, bool variant_w)
{
    if (L.parked.num_units == 0) return hipSuccess;
    ParkedArgs A;
    A.units = L.parked.units; A.layers = L.parked.layers; A.S = S;
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) {
        A.grad[i] = W.grad[i]; A.err[i] = W.err[i]; A.codes[i] = W.codes[i]; A.scales[i] = W.scales[i];
        A.mw[i] = W.mw[i]; A.vw[i] = W.vw[i];
    }
    A.row = L.max_row; A.maxima = L.tile_max + rest_maxima(L.rest);
    A.meeting = L.parked.meeting; A.aside = L.parked.aside; A.meeting_words = L.parked.meeting_words;
    A.inv_scales = L.inv_scales; A.err_bound = L.err_bound; A.bound_factor = residual_bound_factor(S);
    A.num_segments = L.num_segments; A.first_worker = first_worker; A.polls = L.parked.polls;
    A.status = L.status;
    A.num_units = (uint32_t)L.parked.num_units; A.total = A.num_units * (uint32_t)num;
    const bool three = L.parked.longest > kParkedLongest;
    if (S.rounding == 0) launch_parked<0>(A, three, variant_w, L.stream);
    else launch_parked<1>(A, three, variant_w, L.stream);
    return hipGetLastError();
}

// `num`: workers whose maxima one pass left.  parked: variant W, p lies in the error buffer.
static void launch_quantizer(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int worker, int num, bool parked)
{
    WorkerArgs A;
    A.tiles = L.scaled.tiles;
    A.status = L.status; A.S = S;
    A.grad = parked ? nullptr : W.grad[worker];
    A.err = W.err[worker]; A.codes = W.codes[worker]; A.scales = W.scales[worker];
    A.fold = make_fold(L, S, worker, num, parked ? moment_parts(L) : 1);
    A.worker = worker;
    A.seg_len = 0;
    A.items = wave_items(L.scaled.shape, kQuantizeElems);
    launch_quantizer(A, L.stream);
}

hipError_t launch_worker_quantize(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int worker)
{
    if (L.scaled.shape.num_tiles == 0) return hipSuccess;
    launch_quantizer(L, S, W, worker, 1, W.grad[worker] == nullptr);
    return hipGetLastError();
}

static void fill_server_args(ServerArgs& A, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp)
{
    A.S = S; A.sp = sp;
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) { A.codes[i] = W.codes[i]; A.scales[i] = W.scales[i]; }
}

template <int U, int ROUNDING, bool W, bool LONG>
static void launch_server_pieces(const ServerArgs& A, hipStream_t stream)
{
    const dim3 grid = wave_grid(A.items), block(64);
    const unsigned need = U ? 0u : (unsigned)(A.S.num_workers * kServerElems / 32 * A.S.code_bits * 4);
    const unsigned least = server_lds(U != 0, A.S.weight_ef && A.S.k_x >= 0), lds = need > least ? need : least;
    if (A.S.mu_bits == 1) hipLaunchKernelGGL((k_server_step<1, U, ROUNDING, W, LONG>), grid, block, lds, stream, A);
    else if (A.S.mu_bits == 2) hipLaunchKernelGGL((k_server_step<2, U, ROUNDING, W, LONG>), grid, block, lds, stream, A);
    else hipLaunchKernelGGL((k_server_step<3, U, ROUNDING, W, LONG>), grid, block, lds, stream, A);
}

template <int ROUNDING, bool W>
static void launch_server_tiles(ServerArgs& A, const Tile* tiles, const ListShape& shape, hipStream_t stream)
{
    if (shape.num_tiles == 0) return;
    A.tiles = tiles;
    A.items = wave_items(shape, kServerElems);
    if (A.items.cut.part_len > kServerElems) launch_server_pieces<0, ROUNDING, W, true>(A, stream);
    else if (A.S.num_workers == 1) launch_server_pieces<1, ROUNDING, W, false>(A, stream);
    else if (A.S.num_workers == 2) launch_server_pieces<2, ROUNDING, W, false>(A, stream);
    else if (A.S.num_workers == 3) launch_server_pieces<3, ROUNDING, W, false>(A, stream);
    else if (A.S.num_workers == 4) launch_server_pieces<4, ROUNDING, W, false>(A, stream);
    else launch_server_pieces<0, ROUNDING, W, false>(A, stream);
}

// the server's part alone, of every layer: no weight codes
template <bool W>
static hipError_t launch_server_alone(const Launch& L, const StepScalars& S, const WorkerPtrs& W_, const ServerPtrs& sp)
{
    if (L.num_tiles == 0) return hipSuccess;
    ServerArgs A;
    fill_server_args(A, S, W_, sp);
    A.S.k_x = -1;
    if (!server_by_section(L.shape, L.short_layers != nullptr)) {
        launch_server_tiles<0, W>(A, L.tiles, L.shape, L.stream);
        return hipGetLastError();
    }
    launch_server_tiles<0, W>(A, L.scaled.tiles, L.scaled.shape, L.stream);
    const Tile* tiles = L.short_layers;
    for (int k = 0; k < kShortSizes; tiles += L.apart.num[k], ++k)
        launch_server_tiles<0, W>(A, tiles, L.short_shape[k], L.stream);
    return hipGetLastError();
}

hipError_t launch_server_step(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp)
{
    return launch_server_alone<false>(L, S, W, sp);
}

hipError_t launch_server_apply_w(const Launch& L, const StepScalars& S, const WorkerPtrs& W, float* x)
{
    return launch_server_alone<true>(L, S, W, ServerPtrs{x, nullptr, nullptr, nullptr, nullptr});
}

static dim3 flat_grid(int64_t n, int threads, int per_block)
{
    const FlatGrid g = flat_blocks(n, threads, per_block);
    return dim3(g.x, g.y);
}

template <int THREADS, int PIECES>
static void launch_weight_quantizer(const WeightArgs& A, hipStream_t stream)
{
    const dim3 grid = flat_grid(A.n, THREADS, THREADS * PIECES * 4), block(THREADS);
    if (A.S.rounding == 0) hipLaunchKernelGGL((k_weight_quantize<0, THREADS, PIECES>), grid, block, 0, stream, A);
    else hipLaunchKernelGGL((k_weight_quantize<1, THREADS, PIECES>), grid, block, 0, stream, A);
}

// Workgroups of 256 threads with four quads per lane where weights, residual and codes stay in the cache and fill the chip
// with them, else of one wavefront with one.  us, 64 x 1 / 256 x 4: int8 codes, 9 bytes per element, 1 M (2^20) elements
// 3.6 / 4.3, 2 M 5.9 / 4.8, 3 M 7.3 / 5.5, 4 M 9.4 / 8.3, 6 M 12.7 / 12.1, 8 M 17.4 / 16.8, 11.7 M 23.8 / 25.1; int16 without
// error feedback, 10 bytes, 2 M 5.5 / 4.1, 4 M 8.3 / 6.6, 8 M 14.6 / 12.5.
static bool quantize_in_cache(int64_t n, int code_bytes, bool residual)
{
    const int64_t bytes = n * (4 + (residual ? 4 : 0) + code_bytes);
    return bytes >= (int64_t)16 << 20 && bytes <= (int64_t)96 << 20;
}

hipError_t launch_weight_quantize(const Launch& L, const StepScalars& S, const float* x, float* werr, void* wcodes)
{
    if (L.num_params == 0) return hipSuccess;
    WeightArgs A;
    A.S = S; A.x = x; A.werr = werr; A.wcodes = wcodes; A.n = L.num_params;
    if (quantize_in_cache(A.n, S.wcode_bytes, werr != nullptr)) launch_weight_quantizer<256, 4>(A, L.stream);
    else launch_weight_quantizer<64, 1>(A, L.stream);
    return hipGetLastError();
}

template <bool HALF, int CODE_BYTES, int THREADS, int PIECES>
static void launch_decoder(const Launch& L, const DequantArgs& A)
{
    hipLaunchKernelGGL((k_weight_dequantize<HALF, CODE_BYTES, THREADS, PIECES>),
                       flat_grid(A.n, THREADS, THREADS * PIECES * (HALF ? 8 : 4)), dim3(THREADS), 0, L.stream, A);
}

// Workgroups of 256 threads with four pieces per lane where codes and output stay in the memory-side cache, else smaller
// ones.  us, 256 x 4 / the other, outputs in the cache where they fit: int8 to fp32 (256 x 2) 8 M 7.4 / 7.9, 11.7 M
// 9.9 / 10.7, 24 M 20.4 / 19.4, 124 M 115 / 94, 400 M 372 / 302; the others (64 x 1) int8 to binary16 2 M 3.7 / 2.8, 4 M
// 3.7 / 3.9, 11.7 M 6.2 / 8.0, 40 M 20.2 / 21.2, 124 M 60.3 / 59.0, 400 M 197 / 181; int16 to fp32 1 M 2.8 / 2.7, 4 M
// 4.0 / 6.0, 11.7 M 11.7 / 13.5, 40 M 38.8 / 38.6, 400 M 406 / 354; int16 to binary16 4 M 3.8 / 4.0, 8 M 5.1 / 6.1, 11.7 M
// 8.7 / 8.2, 400 M 252 / 237.  Outputs written in turn from one stream, int8 to binary16, 2^21 codes (6 MB): 2.9 / 3.6.
static bool decode_in_cache(int64_t n, int code_bytes, bool half)
{
    const int64_t bytes = n * (code_bytes + (half ? 2 : 4));
    return bytes >= (int64_t)6 << 20 && bytes <= (int64_t)(half && code_bytes == 2 ? 40 : 160) << 20;
}

hipError_t launch_weight_dequantize(const Launch& L, const StepScalars& S, const void* wcodes, void* xhat, bool half)
{
    if (L.num_params == 0) return hipSuccess;
    DequantArgs A;
    A.wcodes = wcodes; A.xhat = xhat; A.n = L.num_params;
    union { uint32_t u; float f; } cv;
    cv.u = (uint32_t)(127 - S.k_x - 1) << 23;
    A.inv_two_kx1 = cv.f;
    const bool cached = decode_in_cache(A.n, S.wcode_bytes, half);
    if (S.wcode_bytes == 1) {
        if (half) cached ? launch_decoder<true, 1, 256, 4>(L, A) : launch_decoder<true, 1, 64, 1>(L, A);
        else cached ? launch_decoder<false, 1, 256, 4>(L, A) : launch_decoder<false, 1, 256, 2>(L, A);
    } else {
        if (half) cached ? launch_decoder<true, 2, 256, 4>(L, A) : launch_decoder<true, 2, 64, 1>(L, A);
        else cached ? launch_decoder<false, 2, 256, 4>(L, A) : launch_decoder<false, 2, 64, 1>(L, A);
    }
    return hipGetLastError();
}

// Two code buffers that overlap would not survive until the server reads them; the main pass reads none.
// Where the buffers lie as qadam_arena_layout deals them and its groups are a third of the device's memory apart or more, the
// streams of the main pass are spread as well as they can be, and from three workers on (variant W: always) it is as fast or
// faster.  ms per step, main pass / by worker, groups 132 GiB apart: 1.3 G parameters, one worker 11.12 / 11.03, two 15.06 / 15.09,
// four 20.13 / 20.44, eight 33.66 / 34.28, variant W 11.00 / 11.20, 18.52 / 18.79, 33.46 / 34.05, 64.08 / 65.19; 24 M, eight 0.657 /
// 0.667; 96 M, three 1.268 / 1.284, eight 2.565 / 2.544; 64 M, four 1.014 / 1.013; 256 M, one 2.15 / 2.07, sixteen 12.48 / 12.53.
// 50 GiB apart: 96 M, eight 2.802 / 2.570; 256 M, sixteen 13.68 / 12.76; 70 GiB: 1.3 G, four 22.24 / 21.01.  Allocated one by one:
// 1.3 G, four 23.05 / 21.49, eight 34.73 / 34.84.
constexpr int64_t kGroupsApart = (int64_t)96 << 30;

static bool dealt_apart(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp, bool variant_w)
{
    const uint64_t big = arena_round((uint64_t)L.num_params * 4u), code = arena_round((uint64_t)L.code_words * 4u);
    auto bytes = [&](Buffer b) {
        return b == Buffer::codes ? code : b == Buffer::wcodes ? arena_round((uint64_t)L.num_params * S.wcode_bytes)
             : b == Buffer::scales ? arena_round((uint64_t)L.num_segments * 4u) : big;
    };
    auto at = [&](Buffer b, int i) -> uint64_t {
        switch (b) {
        case Buffer::x: return (uint64_t)sp.x;
        case Buffer::m: return (uint64_t)sp.m;
        case Buffer::v: return (uint64_t)sp.v;
        case Buffer::werr: return (uint64_t)sp.werr;
        case Buffer::err: return (uint64_t)W.err[i];
        case Buffer::mw: return (uint64_t)W.mw[i];
        case Buffer::vw: return (uint64_t)W.vw[i];
        case Buffer::grad: return (uint64_t)W.grad[i];
        default: return 0;                          // the small ones may lie anywhere
        }
    };
    return groups_apart(S.num_workers, variant_w, bytes, at) >= kGroupsApart;
}

bool step_by_worker(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp, bool variant_w)
{
    if (L.parked_done) return true;
    if (!worth_by_worker(L.scaled.num_elems, L.off_grid_elems, S.num_workers, variant_w, S.rounding == 1)) return false;
    if ((variant_w || S.num_workers > 2) && dealt_apart(L, S, W, sp, variant_w)) return false;
    return !codes_overlap(L, W, 0, S.num_workers);
}

static void launch_by_worker(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp, bool variant_w)
{
    if (L.scaled.shape.num_tiles > 0)
        for (int i = 0; i < S.num_workers; ++i) launch_quantizer(L, S, W, i, S.num_workers, variant_w);
    ServerArgs A;
    fill_server_args(A, S, W, sp);
    if (S.rounding == 0) {
        if (variant_w) launch_server_tiles<0, true>(A, L.served_tiles, L.served, L.stream);
        else launch_server_tiles<0, false>(A, L.served_tiles, L.served, L.stream);
    } else {
        if (variant_w) launch_server_tiles<1, true>(A, L.served_tiles, L.served, L.stream);
        else launch_server_tiles<1, false>(A, L.served_tiles, L.served, L.stream);
    }
}

// LDS that a workgroup of the main pass reserves and does not use: it holds the pass to 16 wavefronts per CU, each
// with the loads of four workers in flight.  More of them only spread the accesses over more DRAM pages, fewer
// leave the memory idle (1.3 G parameters, 4 workers, whole step: 20 per CU 22.0 ms, 16 21.7, 12 21.6, 8 22.5;
// 124 M, 8 workers: 3.95 / 3.89 / 3.87 / 4.09; 11.7 M, 4 workers: 229 / 227 / 236 / 250 us).  Variant W, which has one load
// per worker in flight where the other has two, reserves none (16 wavefronts / as many as fit, 28: 1.3 G, 8 workers, the pass
// 18.99 / 17.41 ms; whole step of 4 workers, 11.7 M 327 / 316 us, 24 M 702 / 681, 64 M 1821 / 1768).
constexpr unsigned kMainPassLds = 10240;

static hipError_t launch_fused_any(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp,
                                   bool variant_w)
{
    if (L.served.num_tiles == 0) return hipSuccess;
    if (step_by_worker(L, S, W, sp, variant_w)) {
        launch_by_worker(L, S, W, sp, variant_w);
        return hipGetLastError();
    }
    FusedArgs A;
    A.tiles = L.scaled.tiles;
    A.status = L.status; A.S = S; A.sp = sp;
    A.fold = make_fold(L, S, 0, S.num_workers, variant_w ? moment_parts(L) : 1);
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) {
        A.grad[i] = W.grad[i]; A.err[i] = W.err[i]; A.codes[i] = W.codes[i]; A.scales[i] = W.scales[i];
    }
    A.items = wave_items(L.scaled.shape, 256);
    const dim3 grid = wave_grid(A.items), block(64);
    const unsigned lds = variant_w ? 0u : kMainPassLds;
    const bool fold = A.fold.tile_max != nullptr;
#define QADAM_LAUNCH_FUSED(R, WV)                                                                                   \
    do {                                                                                                            \
        if (!fold) hipLaunchKernelGGL((k_fused<R, 4, WV>), grid, block, lds, L.stream, A);                          \
        else if (S.num_workers == 1) hipLaunchKernelGGL((k_fused<R, 1, WV>), grid, block, 0, L.stream, A);          \
        else if (S.num_workers <= 4) hipLaunchKernelGGL((k_fused<R, kFoldFew, WV>), grid, block, 0, L.stream, A);   \
        else hipLaunchKernelGGL((k_fused<R, kFoldMany, WV>), grid, block, 0, L.stream, A);                          \
    } while (0)
    if (S.rounding == 0) {
        if (variant_w) QADAM_LAUNCH_FUSED(0, true); else QADAM_LAUNCH_FUSED(0, false);
    } else {
        if (variant_w) QADAM_LAUNCH_FUSED(1, true); else QADAM_LAUNCH_FUSED(1, false);
    }
#undef QADAM_LAUNCH_FUSED
    return hipGetLastError();
}

template <int ROUNDING, bool SERVER, bool W>
static void launch_layers(LayerArgs& A, const ShortLayers& layers, hipStream_t stream)
{
    for (int k = 0; k < kShortSizes; A.tiles += layers.num[k], ++k) {
        if (layers.num[k] == 0) continue;
        A.items = layer_items(layers.num[k]);
        const dim3 grid = wave_grid(A.items);
        if (k == 0) hipLaunchKernelGGL((k_layers<ROUNDING, 64, 1, SERVER, W>), grid, dim3(64), 0, stream, A);
        else if (k == 1) hipLaunchKernelGGL((k_layers<ROUNDING, 256, 1, SERVER, W>), grid, dim3(256), 0, stream, A);
        else hipLaunchKernelGGL((k_layers<ROUNDING, 256, 4, SERVER, W>), grid, dim3(256), 0, stream, A);
    }
}

template <bool SERVER>
static hipError_t launch_short_layers(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp,
                                      int worker, bool variant_w)
{
    if (!L.short_layers) return hipSuccess;
    LayerArgs A;
    A.tiles = L.short_layers;
    A.status = L.status; A.S = S; A.sp = sp;
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) {
        A.grad[i] = W.grad[i]; A.mw[i] = W.mw[i]; A.vw[i] = W.vw[i];
        A.err[i] = W.err[i]; A.codes[i] = W.codes[i]; A.scales[i] = W.scales[i];
    }
    A.err_bound = L.err_bound; A.bound_factor = residual_bound_factor(S);
    A.first_worker = worker; A.num_segments = L.num_segments;
    if (S.rounding == 0) {
        if (variant_w) launch_layers<0, SERVER, true>(A, L.apart, L.stream);
        else launch_layers<0, SERVER, false>(A, L.apart, L.stream);
    } else {
        if (variant_w) launch_layers<1, SERVER, true>(A, L.apart, L.stream);
        else launch_layers<1, SERVER, false>(A, L.apart, L.stream);
    }
    return hipGetLastError();
}

hipError_t launch_short_layers(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int worker, bool variant_w)
{
    return launch_short_layers<false>(L, S, W, ServerPtrs{}, worker, variant_w);
}

hipError_t launch_short_layers(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp, bool variant_w)
{
    return launch_short_layers<true>(L, S, W, sp, 0, variant_w);
}

hipError_t launch_fused(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp)
{
    return launch_fused_any(L, S, W, sp, false);
}

hipError_t launch_plain_messages(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp,
                                 bool variant_w)
{
    if (L.num_tiles == 0) return hipSuccess;
    FusedArgs A;
    A.tiles = L.tiles; A.items = Items{};
    A.status = L.status; A.fold = Fold{}; A.S = S; A.sp = sp;
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) {
        A.grad[i] = W.grad[i]; A.err[i] = W.err[i]; A.codes[i] = nullptr; A.scales[i] = nullptr;
    }
    const dim3 grid(L.num_tiles), block(kBlockThreads);
    const bool four = S.num_workers % 4 == 0;
#define QADAM_LAUNCH_PLAIN(R, WV)                                                                     \
    do {                                                                                              \
        if (four) hipLaunchKernelGGL((k_plain_messages<R, 4, WV>), grid, block, 0, L.stream, A);      \
        else hipLaunchKernelGGL((k_plain_messages<R, 1, WV>), grid, block, 0, L.stream, A);           \
    } while (0)
    if (S.rounding == 0) {
        if (variant_w) QADAM_LAUNCH_PLAIN(0, true); else QADAM_LAUNCH_PLAIN(0, false);
    } else {
        if (variant_w) QADAM_LAUNCH_PLAIN(1, true); else QADAM_LAUNCH_PLAIN(1, false);
    }
#undef QADAM_LAUNCH_PLAIN
    return hipGetLastError();
}

hipError_t launch_fused_w(const Launch& L, const StepScalars& S, const WorkerPtrs& W, const ServerPtrs& sp)
{
    return launch_fused_any(L, S, W, sp, true);
}

hipError_t launch_layer_sumsq(const Launch& L, const float* a, const float* b, double* out)
{
    if (L.num_segments == 0) return hipSuccess;
    SumsqArgs A;
    A.tiles = L.tiles; A.a = a; A.b = b; A.tile_sum = L.tile_sum; A.seg_tile_begin = L.seg_tile_begin; A.out = out;
    if (L.num_tiles > 0)
        hipLaunchKernelGGL(k_sumsq_tiles, dim3(L.num_tiles), dim3(kBlockThreads), 0, L.stream, A);
    hipLaunchKernelGGL(k_sumsq_layers, dim3(L.num_segments), dim3(kBlockThreads), 0, L.stream, A);
    return hipGetLastError();
}

hipError_t launch_worker_moments_w(const Launch& L, const StepScalars& S, const WorkerPtrs& W, int first_worker, int num)
{
    if (L.scaled.shape.num_tiles == 0 || num == 0) return hipSuccess;
    MomentsWArgs A;
    A.tiles = L.scaled.tiles; A.row = L.max_row; A.S = S;
    for (int i = 0; i < QADAM_MAX_WORKERS; ++i) {
        A.grad[i] = W.grad[i]; A.mw[i] = W.mw[i]; A.vw[i] = W.vw[i]; A.err[i] = W.err[i];
    }
    A.tile_max = L.tile_max;
    A.first_worker = first_worker;
    A.cut = moment_cut(L.scaled.shape);
    const dim3 grid((unsigned)L.scaled.shape.num_tiles * A.cut.parts, num), block(kBlockThreads);
    if (keep_parked(L.scaled.num_elems, num)) hipLaunchKernelGGL(k_moments_w<true>, grid, block, 0, L.stream, A);
    else hipLaunchKernelGGL(k_moments_w<false>, grid, block, 0, L.stream, A);
    return hipGetLastError();
}

// ================================================================================================
// Handle-free quantization of one segment without any allocation.
// The device memory the kernels need beyond the caller's buffers -- one maximum per tile, the
// reciprocal scale, the residual bound and a status word -- is this file-scope array.  Every GPU
// holds its own copy at its own address; host code must never pass the array's name to a kernel
// or a HIP call (on the host it is only a stand-in for the symbol): it uses the address that
// hipGetSymbolAddress returned for the current device.
// ================================================================================================
constexpr int kNoallocMaxTiles = (int)(kNoallocMaxElems / kTileElems);
constexpr int kNoallocExtraWords = 64;      // [0] reciprocal scale, [1] residual bound, [2] status, rest unused
constexpr int kMaxDevices = 64;
static __device__ __align__(256) uint32_t scratch[kNoallocMaxTiles + kNoallocExtraWords];

static uint32_t* g_scratch_ptr[kMaxDevices];          // per device, null until looked up
static std::mutex g_scratch_mutex;

static hipError_t scratch_for_current_device(uint32_t** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<uint32_t*>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t noalloc_prepare()
{
    uint32_t* p = nullptr;
    return scratch_for_current_device(&p);
}

// qadam_worker_quantize for worker 0 of a one-segment vector of n elements: one launch up to kSegmentElems, beyond that
// its two or three, with tile records computed in the kernels and the scratch rows taken from the static array.
// Nothing of the array has to start at zero: every tile maximum, the reciprocal and the bound are
// written before they are read, and the status word is only ever OR-ed into and never read here.
hipError_t noalloc_quantize_segment(const StepScalars& S, int64_t n, const float* grad, float* err, uint32_t* codes,
                                    float* scale_out, hipStream_t stream)
{
    uint32_t* sc = nullptr;
    hipError_t e = scratch_for_current_device(&sc);
    if (e != hipSuccess) return e;
    if (n > 0 && n <= kSegmentElems) {
        SegmentArgs A;
        A.S = S; A.grad = grad; A.err = err; A.codes = codes; A.scale = scale_out; A.n = (int)n;
        hipLaunchKernelGGL(k_segment, dim3(1), dim3(kSegmentThreads), 0, stream, A);
        return hipGetLastError();
    }
    const int num_tiles = (int)((n + kTileElems - 1) / kTileElems);
    uint32_t* tile_max = sc;
    float* inv_scale = reinterpret_cast<float*>(sc + kNoallocMaxTiles);
    float* err_bound = reinterpret_cast<float*>(sc + kNoallocMaxTiles + 1);
    uint32_t* status = sc + kNoallocMaxTiles + 2;

    ListShape shape{};
    if (num_tiles > 0) {
        add_tiles(shape, num_tiles - 1, kTileElems);
        add_tiles(shape, 1, (int)(n - (int64_t)(num_tiles - 1) * kTileElems));
        AmaxArgs A;
        std::memset(&A, 0, sizeof A);
        A.tiles = nullptr; A.num_tiles = num_tiles; A.seg_len = n;
        A.grad[0] = grad; A.err[0] = err;
        A.tile_max = tile_max; A.row = num_tiles; A.first_worker = 0; A.num_segments = 1; A.status = status;
        launch_scan(A, shape, n, 1, stream);
    }
    Fold F;
    std::memset(&F, 0, sizeof F);
    F.row = num_tiles; F.per_tile = 1; F.num_segments = 1;
    F.inv_scales = inv_scale; F.err_bound = err_bound; F.bound_factor = residual_bound_factor(S);
    if (num_tiles > 0 && fold_in_quantizer(num_tiles, n, num_tiles, 1, 1)) {
        F.tile_max = tile_max;
    } else {
        ScaleArgs R;
        std::memset(&R, 0, sizeof R);
        R.scales[0] = scale_out; R.inv_scales = inv_scale; R.tile_max = tile_max; R.seg_tile_begin = nullptr;
        R.first_worker = 0; R.num_segments = 1; R.num_tiles = num_tiles; R.row = num_tiles; R.max_per_tile = 1;
        R.err_bound = err_bound; R.thr = nullptr;
        R.bound_factor = residual_bound_factor(S);
        R.sample_stride = kSampleStride;
        hipLaunchKernelGGL(k_reduce_scales, dim3(1, 1), dim3(kReduceThreads), 0, stream, R);
    }
    if (num_tiles > 0) {
        WorkerArgs W;
        std::memset(&W, 0, sizeof W);
        W.tiles = nullptr; W.seg_len = n;
        W.status = status; W.S = S;
        W.grad = grad; W.err = err; W.codes = codes; W.scales = scale_out; W.fold = F;
        W.worker = 0;
        W.items = wave_items(shape, kQuantizeElems);
        launch_quantizer(W, stream);
    }
    return hipGetLastError();
}

}  // namespace qadam
