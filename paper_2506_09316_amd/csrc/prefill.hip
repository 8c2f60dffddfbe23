// Chunked DSLA prefill for gfx950 (paper Section 4.1: state-update equation and blended
// read-out, evaluated 32 tokens at a time).
//
// The token recurrence is regrouped so that every bracket is a dense contraction and runs on MFMA; the
// algebra is written out above the kernel body ("Chunk algebra").  With Qc = [Q~^1 | Q~^2] and
// Kc = [K~^1 | K~^2] (width 2 d_k) the blend of the two states is part of the contractions:
// scores = Qc Kc^T, carried read-out = Qc [T^1; T^2].
//
// Parallel decomposition.  A sequence is cut into P segments so that B*H*P workgroups fill the
// chip.  (1) segment_state: every segment but the last computes, from a zero state, its state
// contribution U and its total log-decay.  (2) segment_scan: an elementwise scan over segments
// turns these into the true state entering each segment.  (3) chunk_loop: every segment runs the
// fused step loop from its true initial state and writes o; the last segment writes the final
// states.  P = 1 runs (3) alone.  (1) and (3) are one kernel template; for 16-bit inputs and gates at d = 128, (1) has a
// kernel of its own that walks a segment backwards (segment_state_fast_kernel, below the template), and for 32-bit inputs both
// have kernels that are made for the rate of fp32 MFMAs (F32Kern; the template keeps the launches with a beta gate).
// Packed sequences of different lengths, if any of them is cut: a one-workgroup kernel turns their offsets into the lists of
// segments that (1) and (3) take their work from, so that no workgroup has a segment that does not exist.  Either every sequence is
// cut, into segments of one length (segment_list), or only the long ones are, from their ends (long_segment_list).  Sequences may be a subset of the packed batch and
// their states entries of a pool (both through index arrays).  Gates arrive as log-gates or as the
// pre-activations of a temperature-sigmoid, which the producers then apply themselves.
//
// Workgroup = D/8 wavefronts (D = d_k = d_v): D/32 consumers and D/32 producers, see "Workgroup layout".
// Consumer w owns state columns [32w, 32w+32) of both states for all d_k rows, as fp32 MFMA accumulators
// (tiles with m = state row, n = column).  Because an MFMA accumulator tile and an MFMA input fragment both
// index lanes by the tile column, those accumulators are fed back as the input fragment of the carried
// read-out without passing through LDS; the partner operand is stored in LDS with the matching order of
// the contraction index (bits 2 and 3 of the feature index swapped).
#include <cstdio>
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "prefill_common.h"

namespace dsla {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------------------------
// Arithmetic-type policies: how a contraction operand is stored in LDS and fed to MFMA.
// A "fragment" is the 8 contraction-index values one lane supplies for a block of 16 contraction
// indices (lane group g = lane/32 supplies indices 8g..8g+7 of the block).
// ---------------------------------------------------------------------------------------------
struct ArithBf16 {
    static constexpr int ESZ = 2;  // bytes per LDS element
    struct Frag {
        bf16x8 v;
    };
    struct Row8 {   // 8 operand values of one token, packed
        u32x4 u;
    };
    static __device__ __forceinline__ Frag load_frag(uint32_t a)
    {
        Frag f;
        f.v = __builtin_bit_cast(bf16x8, lds_ld<u32x4>(a));
        return f;
    }
    // Two transposing 8-byte reads (see Kern::consume): contraction positions 0..3 from address a, 4..7 from a + step.
    static __device__ __forceinline__ Frag load_frag_tr(uint32_t a, uint32_t step)
    {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<s16x4 DSLA_LDS *>(static_cast<uintptr_t>(a)));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<s16x4 DSLA_LDS *>(static_cast<uintptr_t>(a + step)));
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        Frag f;
        f.v = __builtin_bit_cast(bf16x8, u32x4{l2[0], l2[1], h2[0], h2[1]});
        return f;
    }
    static __device__ __forceinline__ uint32_t pack2(float a, float b)
    {
        f32x2 x = {a, b};
        bf16x2 y = __builtin_convertvector(x, bf16x2);
        return __builtin_bit_cast(uint32_t, y);
    }
    static __device__ __forceinline__ Row8 pack_row(const float (&x)[8])
    {
        Row8 r;
        r.u = u32x4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7])};
        return r;
    }
    static __device__ __forceinline__ void store_row(uint32_t a, const Row8 &r) { lds_st<u32x4>(a, r.u); }
    static constexpr uint32_t kSignBits = 0x80008000u;   // sign bits of the two values of a packed word
    static __device__ __forceinline__ Row8 flip_sign(Row8 r, uint32_t bits)   // bits: kSignBits or 0
    {
        r.u ^= u32x4{bits, bits, bits, bits};
        return r;
    }
    // element e of RPT consecutive tokens -> RPT adjacent LDS elements
    template <int RPT>
    static __device__ __forceinline__ void store_tokens(uint32_t a, const Row8 (&r)[RPT], int e)
    {
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
        const uint32_t lo = __builtin_amdgcn_perm(r[1].u[e >> 1], r[0].u[e >> 1], sel);
        if constexpr (RPT == 4) {
            const uint32_t hi = __builtin_amdgcn_perm(r[3].u[e >> 1], r[2].u[e >> 1], sel);
            lds_st<u32x2>(a, u32x2{lo, hi});
        } else {
            lds_st<uint32_t>(a, lo);
        }
    }
    static __device__ __forceinline__ void store4(uint32_t a, float x0, float x1, float x2, float x3)
    {
        lds_st<u32x2>(a, u32x2{pack2(x0, x1), pack2(x2, x3)});
    }
    static __device__ __forceinline__ f32x4 load4(uint32_t a)   // four adjacent operand elements
    {
        const u32x2 u = lds_ld<u32x2>(a);
        return f32x4{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16),
                     __uint_as_float(u[1] & 0xffff0000u)};
    }
    static __device__ __forceinline__ Frag from_acc(const f32x16 &acc, int half)
    {
        const u32x4 u = {pack2(acc[8 * half + 0], acc[8 * half + 1]), pack2(acc[8 * half + 2], acc[8 * half + 3]),
                         pack2(acc[8 * half + 4], acc[8 * half + 5]), pack2(acc[8 * half + 6], acc[8 * half + 7])};
        Frag f;
        f.v = __builtin_bit_cast(bf16x8, u);
        return f;
    }
    static __device__ __forceinline__ void mma(f32x16 &acc, const Frag &a, const Frag &b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, acc, 0, 0, 0);
    }
};

struct ArithF32 {
    static constexpr int ESZ = 4;
    struct Frag {
        float v[8];
    };
    struct Row8 {
        float x[8];
    };
    static __device__ __forceinline__ Frag load_frag(uint32_t a)
    {
        const f32x4 lo = lds_ld<f32x4>(a), hi = lds_ld<f32x4>(a + 16);
        Frag f;
        f.v[0] = lo[0]; f.v[1] = lo[1]; f.v[2] = lo[2]; f.v[3] = lo[3];
        f.v[4] = hi[0]; f.v[5] = hi[1]; f.v[6] = hi[2]; f.v[7] = hi[3];
        return f;
    }
    static __device__ __forceinline__ Frag load_frag_tr(uint32_t, uint32_t) { return Frag{}; }   // 16-bit storage only
    static __device__ __forceinline__ Row8 pack_row(const float (&x)[8])
    {
        Row8 r;
#pragma unroll
        for (int e = 0; e < 8; ++e) r.x[e] = x[e];
        return r;
    }
    static __device__ __forceinline__ void store_row(uint32_t a, const Row8 &r)
    {
        lds_st<f32x4>(a, f32x4{r.x[0], r.x[1], r.x[2], r.x[3]});
        lds_st<f32x4>(a + 16, f32x4{r.x[4], r.x[5], r.x[6], r.x[7]});
    }
    static constexpr uint32_t kSignBits = 0x80000000u;
    static __device__ __forceinline__ Row8 flip_sign(Row8 r, uint32_t bits)   // bits: kSignBits or 0
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) r.x[e] = __uint_as_float(__float_as_uint(r.x[e]) ^ bits);
        return r;
    }
    template <int RPT>
    static __device__ __forceinline__ void store_tokens(uint32_t a, const Row8 (&r)[RPT], int e)
    {
        if constexpr (RPT == 4)
            lds_st<f32x4>(a, f32x4{r[0].x[e], r[1].x[e], r[2].x[e], r[3].x[e]});
        else
            lds_st<f32x2>(a, f32x2{r[0].x[e], r[1].x[e]});
    }
    static __device__ __forceinline__ void store4(uint32_t a, float x0, float x1, float x2, float x3)
    {
        lds_st<f32x4>(a, f32x4{x0, x1, x2, x3});
    }
    static __device__ __forceinline__ f32x4 load4(uint32_t a) { return lds_ld<f32x4>(a); }
    static __device__ __forceinline__ Frag from_acc(const f32x16 &acc, int half)
    {
        Frag f;
#pragma unroll
        for (int e = 0; e < 8; ++e) f.v[e] = acc[8 * half + e];
        return f;
    }
    // 32x32x2 fp32 MFMA: lane group g supplies one contraction index per instruction.
    static __device__ __forceinline__ void mma(f32x16 &acc, const Frag &a, const Frag &b)
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.v[e], b.v[e], acc, 0, 0, 0);
    }
};

template <class TIO>
using ArithOf = typename std::conditional<std::is_same<TIO, bf16_t>::value, ArithBf16, ArithF32>::type;

// ---- raw global loads (kept unconverted while in flight); address = uniform base + 32-bit lane offset ----
template <class T>
struct Raw8;
template <>
struct Raw8<bf16_t> {
    u32x4 u;
    __device__ __forceinline__ void load(const bf16_t *base, uint32_t elem_off)
    {
        u = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(base) + elem_off * 2u);
    }
    __device__ __forceinline__ void zero() { u = u32x4{0, 0, 0, 0}; }
    __device__ __forceinline__ void fill_huge() { u = u32x4{0x7e007e00u, 0x7e007e00u, 0x7e007e00u, 0x7e007e00u}; }   // 2^125
    // orders every later use of the loaded value after `dep` has been computed (no instruction is emitted)
    __device__ __forceinline__ void pin_after(float dep) { asm volatile("" : "+v"(u) : "v"(dep)); }
    __device__ __forceinline__ void unpack(float (&f)[8]) const
    {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            f[2 * w] = __uint_as_float(u[w] << 16);
            f[2 * w + 1] = __uint_as_float(u[w] & 0xffff0000u);
        }
    }
};
template <>
struct Raw8<float> {
    f32x4 a, b;
    __device__ __forceinline__ void load(const float *base, uint32_t elem_off)
    {
        const char *p = reinterpret_cast<const char *>(base) + elem_off * 4u;
        a = *reinterpret_cast<const f32x4 *>(p);
        b = *reinterpret_cast<const f32x4 *>(p + 16);
    }
    __device__ __forceinline__ void zero() { a = b = f32x4{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ void fill_huge() { a = b = f32x4{0x1p125f, 0x1p125f, 0x1p125f, 0x1p125f}; }
    __device__ __forceinline__ void pin_after(float dep) { asm volatile("" : "+v"(a), "+v"(b) : "v"(dep)); }
    __device__ __forceinline__ void unpack(float (&f)[8]) const
    {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            f[w] = a[w];
            f[4 + w] = b[w];
        }
    }
};
template <class T>
struct Raw4;
template <>
struct Raw4<bf16_t> {
    u32x2 u;
    __device__ __forceinline__ void load(const bf16_t *base, uint32_t elem_off)
    {
        u = *reinterpret_cast<const u32x2 *>(reinterpret_cast<const char *>(base) + elem_off * 2u);
    }
    __device__ __forceinline__ void zero() { u = u32x2{0, 0}; }
};
template <>
struct Raw4<float> {
    f32x4 a;
    __device__ __forceinline__ void load(const float *base, uint32_t elem_off)
    {
        a = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const char *>(base) + elem_off * 4u);
    }
    __device__ __forceinline__ void zero() { a = f32x4{0.f, 0.f, 0.f, 0.f}; }
};

// Transposed store of V: element e (0..3) of RPT consecutive tokens -> RPT adjacent LDS elements.
// bf16 data is moved with byte permutes (no conversion); fp32 data is stored as is.
template <int RPT>
__device__ __forceinline__ void store_v_tokens(uint32_t a, const Raw4<bf16_t> (&v)[RPT], int e)
{
    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
    const uint32_t lo = __builtin_amdgcn_perm(v[1].u[e >> 1], v[0].u[e >> 1], sel);
    if constexpr (RPT == 4) {
        const uint32_t hi = __builtin_amdgcn_perm(v[3].u[e >> 1], v[2].u[e >> 1], sel);
        lds_st<u32x2>(a, u32x2{lo, hi});
    } else {
        lds_st<uint32_t>(a, lo);
    }
}
template <int RPT>
__device__ __forceinline__ void store_v_tokens(uint32_t a, const Raw4<float> (&v)[RPT], int e)
{
    if constexpr (RPT == 4)
        lds_st<f32x4>(a, f32x4{v[0].a[e], v[1].a[e], v[2].a[e], v[3].a[e]});
    else
        lds_st<f32x2>(a, f32x2{v[0].a[e], v[1].a[e]});
}

template <int RPT>
__device__ __forceinline__ void store_v_tokens(uint32_t a, const Raw8<bf16_t> (&v)[RPT], int e)
{
    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
    const uint32_t lo = __builtin_amdgcn_perm(v[1].u[e >> 1], v[0].u[e >> 1], sel);
    if constexpr (RPT == 4) {
        const uint32_t hi = __builtin_amdgcn_perm(v[3].u[e >> 1], v[2].u[e >> 1], sel);
        lds_st<u32x2>(a, u32x2{lo, hi});
    } else {
        lds_st<uint32_t>(a, lo);
    }
}
template <int RPT>
__device__ __forceinline__ void store_v_tokens(uint32_t a, const Raw8<float> (&v)[RPT], int e)
{
    auto pick = [&](const Raw8<float> &r) -> float { return e < 4 ? r.a[e & 3] : r.b[e & 3]; };
    if constexpr (RPT == 4)
        lds_st<f32x4>(a, f32x4{pick(v[0]), pick(v[1]), pick(v[2]), pick(v[3])});
    else
        lds_st<f32x2>(a, f32x2{pick(v[0]), pick(v[1])});
}

// a loaded row piece of V as it is (16-bit storage only)
__device__ __forceinline__ void store_v_row(uint32_t a, const Raw8<bf16_t> &v) { lds_st<u32x4>(a, v.u); }

// four adjacent output elements -> global
__device__ __forceinline__ void store4_global(bf16_t *p, float a, float b, float c, float d)
{
    *reinterpret_cast<u32x2 *>(p) = u32x2{ArithBf16::pack2(a, b), ArithBf16::pack2(c, d)};
}
__device__ __forceinline__ void store4_global(float *p, float a, float b, float c, float d)
{
    *reinterpret_cast<f32x4 *>(p) = f32x4{a, b, c, d};
}

// Keeps the computation of x where it stands.  Without it the compiler gathers the MFMAs of one accumulator and lets each wait for
// an LDS read that it issues right before (scheduling barriers alone come too late: the order is gone before they count, and the
// fragments kept for later spill 112 registers).  A step of a consumer alone 2.1 -> 1.2 us, registers 255 -> 235; the producers, 1.9 us,
// bound a step then as before: 8 x 8192 tokens 711 -> 701 us, 16384 tokens 273.7 -> 270.7, 1000 on carried states 49.9 -> 49.4.  At d = 64 two
// workgroups share a compute unit and the compiler's order is the better one (32 heads of 2000 tokens 39.2, this 40.4).
__device__ __forceinline__ void stay(f32x16 &x) { asm volatile("" : "+v"(x) : : "memory"); }

// Software-pipelined sequence of N steps: the LDS fragment of step s + DEPTH is requested before the
// MFMA of step s is issued, so that LDS latency overlaps DEPTH matrix instructions.  Fully unrolled.
// kTr: the fragments come from rows by two transposing reads, the second TR_STEP bytes (two row slots) further.
// kStay: the steps stay in this order (with stay() in each of them).
template <int N, int DEPTH, class ARITH, bool kTr = false, bool kStay = false, class AddrF, class StepF>
__device__ __forceinline__ void pipelined_steps(AddrF addr, StepF step, uint32_t tr_step = 0)
{
    auto load = [&](int i) { return kTr ? ARITH::load_frag_tr(addr(i), tr_step) : ARITH::load_frag(addr(i)); };
    typename ARITH::Frag buf[DEPTH];
#pragma unroll
    for (int i = 0; i < DEPTH && i < N; ++i) buf[i] = load(i);
#pragma unroll
    for (int s = 0; s < N; ++s) {
        const typename ARITH::Frag cur = buf[s % DEPTH];
        if (s + DEPTH < N) buf[s % DEPTH] = load(s + DEPTH);
        step(s, cur);
        if constexpr (kStay) __builtin_amdgcn_sched_barrier(0);
    }
}

// ---------------------------------------------------------------------------------------------
// Workgroup layout: producer / consumer wavefronts.  4 D threads = D/8 wavefronts.  The first D/32
// wavefronts are CONSUMERS: wavefront ct owns columns [32 ct, 32 ct + 32) of BOTH states for all d_k rows as fp32
// MFMA accumulators and runs every contraction of a step.  The other D/32 wavefronts are PRODUCERS: they load
// the inputs of later steps, run the gate scan and write the contraction operands of the NEXT step into the
// other half of a double-buffered LDS.  One workgroup barrier per step hands a finished operand set from the
// producers to the consumers.  Each SIMD hosts one consumer and one producer wavefront, so the VALU-bound
// preparation and the MFMA-bound contractions of neighbouring steps overlap.  A step is S = 32 tokens (a chunk
// of 64 is two steps): two operand sets of 32 tokens fit in the 160 KB LDS, two sets of 64 do not.
//
// Step algebra (Section 4.1 unrolled over the S = 32 tokens of a step).  Per state and feature: b_s = log2 of the gate
// product from the first token of the step up to and including token s (b_s <= 0), R = -b_31 the log2 decay of the whole
// step, and c_s = b_s + R/2 the same exponent centred on the step, so that |c_s| <= R/2.  T = the state in the frame of
// the middle of the step, T = 2^{-R/2} S at the start of the step:
//     Q~ = gamma_i scale q 2^{c}             K~ = k 2^{-c}                 (factors between 2^{-R/2} and 2^{+R/2})
//     o  =  Q~ T  +  mask_{key <= query}(Q~ K~^T) V                        (both states in one contraction of width 2 d_k)
//     T <-  T + K~^T V
//   between two steps the state moves from one middle frame to the next, at the end of a segment to its own frame:
//     T <-  diag(2^{-(R + R_next)/2}) T          (R_next = 0 after the last step; past 2^-120 as two factors)
//   (the 16-bit step loop leaves the frame where it is for several steps while the exponents stay small: line_scan_b)
// Centring halves the largest exponent a step can produce: the factors stay finite while R < 2 * 115, and nothing
// links the exponents of different steps.
//
// Beta mode (Kern<.., kBeta = true>, extended launches only): ONE state with the outer-product gate alpha^T beta of the
// background section on gated linear attention, S[d][j] <- alpha[d] beta[j] S[d][j] + k[d] v[j].  The tensor g1 holds
// log alpha as usual, g2 holds log beta (one value per token and COLUMN), S1 is the state, S2 is not used.  The decay
// along the columns is split like the one along the rows: with c' the centred cumulative log2 beta of a step,
//     V~ = v 2^{-c'}        o = 2^{+c'} . (Q~ T + mask(Q~ K~^T) V~)        T <- T + K~^T V~
// and T lives in the middle frame of the step for rows and columns alike.  The machinery of the second state carries
// beta: its gate scan gives c', its Q~ slot in LDS holds the output factors 2^{c'}, its slot of frame changes those of
// the columns; its K~ and its half of the contractions do not exist.
template <int D, class TIO, class TG, bool kFull, bool kExt = false, bool kBeta = false>
struct Kern {
    static_assert(kExt || !kBeta, "beta mode is an extended launch");
    static constexpr int NST = kBeta ? 1 : 2;   // states in the contractions
    using A = ArithOf<TIO>;
    using Frag = typename A::Frag;
    using Row8 = typename A::Row8;
    static constexpr int ESZ = A::ESZ;

    static constexpr int S = 32;            // tokens per step
    static constexpr int CT = D / 32;       // column tiles = consumer wavefronts = producer wavefronts
    static constexpr int NW = 2 * CT;       // wavefronts
    static constexpr int NT = 64 * NW;      // threads (= 4 D)
    static constexpr int SGN = 16;          // token pairs per step
    static constexpr int RPT = 2;           // tokens per producer thread
    static constexpr int QP = 2 * D + 8;    // pitch of row-layout operands (elements)
    // Token-contiguous operands (Kt, Vt): a row holds the S tokens of one feature (column) as 4 pieces of 8 tokens,
    // without padding; piece c of row R sits at piece position c ^ ((R / 2) % 4), so that the 8 rows a group of 8
    // lanes reads with one 16-byte access each fall into 8 different bank groups.
    static constexpr int TP = S;            // pitch of token-contiguous operands (elements)
    static __device__ __forceinline__ uint32_t tpiece(uint32_t piece, uint32_t row) { return piece ^ ((row >> 1) & 3u); }
    static constexpr int DT = D / 32;       // 32-row tiles of a state
    static constexpr int KB = S / 16;       // contraction blocks over tokens
    static constexpr int NK = 2 * D / 16;   // contraction blocks over the 2 d_k features

    // LDS map (bytes).  Two operand sets; per set:
    static constexpr uint32_t O_QS = 0;                                        // [token][i*D + d]            Q'
    // K~: 16-bit storage keeps ONE copy, in rows [token][i*D + d] of pitch QP; the consumers read it as rows (scores)
    // and, for the update, transposed with ds_read_b64_tr_b16.  Token t sits in row slot kslot(t): the two low bit pairs
    // of the token index swapped.  The 16 rows that 16 lanes read at the same feature then lie in 16 different slots
    // (each slot shifts the banks by 16 bytes: pitch), and the 4 consecutive tokens a pass of the transposing read
    // takes 64 bytes each from lie 4 slots apart: 64 bytes apart in the banks.  32-bit storage keeps two copies: rows
    // (step loop only) and the token-contiguous one [i*D + rho(d)][rho(token)].
    // (Step loop only: in the segment pre-pass, whose consumers have little else to do, the doubled number of LDS read
    // instructions gets in the way of the producers' gate scan, which is bound by its LDS round trips: 119.6 against
    // 116.8 us.)
    static constexpr bool kTrK = ESZ == 2 && kFull;
    static __device__ __forceinline__ uint32_t kslot(uint32_t t) { return (t & ~15u) | ((t & 3u) << 2) | ((t >> 2) & 3u); }
    static constexpr uint32_t O_KS = O_QS + (kFull ? S * QP * ESZ : 0);
    static constexpr uint32_t O_KT = O_KS + ((kFull || kTrK) ? S * QP * ESZ : 0);
    // V: 16-bit storage keeps the rows as loaded, [token][column] without padding, the 64-byte quarter q of row r at
    // quarter position q ^ vswz(r), and the consumers read them with the transposing LDS read, a pass of which takes one
    // quarter from each of 4 consecutive rows: they fall into different banks.  32-bit storage keeps the
    // token-contiguous copy [column][rho(token)].  Both take S * D elements.
    static constexpr bool kTrV = ESZ == 2;
    static __device__ __forceinline__ uint32_t vswz(uint32_t row) { return D == 128 ? (row & 3u) : ((row >> 1) & 1u); }
    static constexpr uint32_t O_VT = O_KT + (kTrK ? 0 : 2 * D * TP * ESZ);
    static constexpr uint32_t O_DEC = O_VT + D * TP * ESZ;                     // float [2D]  frame change after the step
    static constexpr uint32_t O_FLAG = O_DEC + 2 * D * 4;                      // uint8 [CT]: per producer wavefront, how often its factors are multiplied in (kLineProd: 0 .. 2) / whether O_DEC2 holds any
    static constexpr uint32_t O_DEC2 = O_FLAG + 16;                            // float [2D] (not kLineProd)  the rest of a frame change beyond one factor
    static constexpr uint32_t SET_BYTES = O_DEC2 + (ESZ == 2 && kFull && !kExt ? 0 : 2 * D * 4);
    static constexpr uint32_t LDS_MAX = 160 * 1024;                            // LDS of a gfx950 compute unit
    // Two operand sets where they fit (the producers then run a whole step ahead of the consumers); one set
    // otherwise (fp32 at d = 128): the producers then only load ahead and prepare between two barriers.
    static constexpr int SETS = (2 * SET_BYTES + CT * 4096 <= LDS_MAX) ? 2 : 1;
    static constexpr uint32_t O_CS = SETS * SET_BYTES;                         // per producer wavefront: float [2][16][32]
    // Output staging (16-bit io only): two buffers of S rows of d_v elements.  The consumers leave the output tile of
    // a step here and write it to memory one step later as whole rows (a row is then complete: it has passed the
    // barrier), which is what the memory system wants; 8-byte pieces straight from the accumulators cost a quarter
    // of the kernel time.
    static constexpr uint32_t O_ENT = O_CS + CT * 4096;                        // float [2D]  frame change into the first step
    static constexpr uint32_t LDS_NOSTAGE = O_ENT + 2 * D * 4, LDS_STAGE = LDS_NOSTAGE + 2 * S * D * ESZ;
    static constexpr bool kStage =   // only where it does not cost a resident workgroup
        kFull && ESZ == 2 && LDS_STAGE <= LDS_MAX && LDS_MAX / LDS_STAGE == LDS_MAX / LDS_NOSTAGE;
    static constexpr uint32_t O_ST = LDS_NOSTAGE;
    static constexpr uint32_t ST_BYTES = S * D * ESZ;
    static constexpr int NC = D * ESZ / 16;                                    // 16-byte pieces per output row
    static constexpr uint32_t LDS_BYTES = O_ST + (kStage ? 2 * ST_BYTES : 0);
    static_assert(LDS_BYTES <= LDS_MAX, "LDS budget");

    // rho: bits 2 and 3 of an index swapped.  Features are stored in Kt rows in rho order and tokens in Kt / Vt
    // columns in rho order.  With this order the 8 accumulator registers of one half of a 32x32 MFMA result tile
    // (lane group g holds tile rows 8a + 4g + b) are exactly the 8 contraction indices lane group g supplies in an
    // MFMA input fragment read from 8 consecutive positions, so results are fed back as inputs without LDS.
    static __device__ __forceinline__ uint32_t rho(uint32_t x) { return (x & ~12u) | ((x & 4u) << 1) | ((x & 8u) >> 1); }

    // Inputs of one step as loaded (unconverted): this thread's 2 tokens x 8 features.
    struct RawIO {
        Raw8<TIO> q[RPT], k[RPT], v[RPT];
    };
    struct RawGates {
        Raw8<TG> g1[RPT], g2[RPT];
    };
    // Where a producer lane reads a step from.  Loads are never predicated (the number of loads in flight stays
    // a compile-time fact, so waiting for the oldest never waits for the newest): a step past the end of the
    // segment re-reads the last one and a token past the end re-reads the last token; the producer zeroes those.
    struct StepSrc {
        const TIO *q, *k, *v;   // uniform: first token of the step, this (batch, head)
        const TG *g1, *g2;
        uint32_t off[RPT];      // per lane: element offset of token 2 sg + j, features 32 pw + 8 dgl ..
        uint32_t offkv[RPT];    // the same inside k and v when they have fewer heads (kExt only)
        __device__ __forceinline__ uint32_t kv(int j) const { return kExt ? offkv[j] : off[j]; }
    };
    static __device__ __forceinline__ void load_gates(RawGates &g, const StepSrc &s)
    {
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            g.g1[j].load(s.g1, s.off[j]);
            g.g2[j].load(s.g2, s.off[j]);
        }
    }
    static __device__ __forceinline__ void load_io(RawIO &r, const StepSrc &s)
    {
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            r.k[j].load(s.k, s.kv(j));
            if (kFull) r.q[j].load(s.q, s.off[j]);
            r.v[j].load(s.v, s.kv(j));
        }
    }
    // The loads a producer issues while it prepares step m, one at a time between its stages: q, k, v of step
    // m + 1 and the gates of step m + 3.  Slot numbers are constants after unrolling.
    struct NoLoads {
        __device__ __forceinline__ void at(int) const {}
    };
    struct NextLoads {
        RawIO &r;
        const StepSrc &rs;
        RawGates &g;
        const StepSrc &gs;
        __device__ __forceinline__ void at(int slot) const
        {
            if (slot == 0) g.g1[0].load(gs.g1, gs.off[0]);
            if (slot == 1) g.g1[1].load(gs.g1, gs.off[1]);
            if (slot == 2) g.g2[0].load(gs.g2, gs.off[0]);
            if (slot == 3) g.g2[1].load(gs.g2, gs.off[1]);
            if (slot == 4) r.k[0].load(rs.k, rs.kv(0));
            if (slot == 5) r.k[1].load(rs.k, rs.kv(1));
            if (slot == 6 && kFull) r.q[0].load(rs.q, rs.off[0]);
            if (slot == 7 && kFull) r.q[1].load(rs.q, rs.off[1]);
            if (slot == 8) r.v[0].load(rs.v, rs.kv(0));
            if (slot == 9) r.v[1].load(rs.v, rs.kv(1));
        }
    };

    // wavefront-private LDS hand-over: the LDS pipeline runs the requests of one wavefront in order; only the
    // compiler has to be kept from moving accesses across
    static __device__ __forceinline__ void wave_sync() { asm volatile("" ::: "memory"); }

    // Per-lane LDS addresses of a producer (operand set 0; a set adds SET_BYTES), computed once.
    // Lane (sg, dgl) of producer wavefront pw handles tokens 2sg, 2sg+1 and features 32 pw + 8 dgl .. + 7 of both
    // states (and the same columns of v); for the scan over tokens lane l owns column (state l/32, feature l%32).
    struct ProdAddr {
        uint32_t tot;   // scan scratch [state][sg][feature]: this lane's 8 features of state 0 (state 1: + 2048)
        uint32_t col;   // scan scratch: this lane's column, token pair 0
        uint32_t dec;   // decay factor of this lane's column
        uint32_t flag;  // does the change of any of this wavefront's columns take a second factor
        uint32_t row;   // row-layout operands: token 2sg, element f0 (token + 1: + QP, state 1: + D elements)
        uint32_t kt[2];   // Kt: row of feature e = 0 of state 0, position of tokens 2sg, 2sg+1; [x]: for features e with (e/2)%2 = x
        uint32_t vt[4];   // Vt: row of column f0, position of tokens 2sg, 2sg+1; [x]: for columns e with (e/2)%4 = x
        uint32_t vrow[RPT];   // V rows (16-bit storage): token 2sg + j, this lane's 8 columns
        uint32_t krow[RPT];   // K~ rows (16-bit storage): row slot of token 2sg + j, element f0 (state 1: + D elements)
        uint32_t sg;
        uint32_t state;   // state of the column this lane scans
        bool preact;      // the gate tensors hold pre-activations, not log-gates (uniform)
        float unit;       // gate sums times this = log2 of the decay: log2 e for log-gates, 1 / tau for pre-activations
        __device__ __forceinline__ ProdAddr(uint32_t sm, int pw, uint32_t lane)
        {
            sg = lane >> 2;
            state = lane >> 5;
            const uint32_t dgl = lane & 3, f0 = 32 * pw + 8 * dgl;
            const uint32_t csw = sm + O_CS + pw * 4096;
            tot = csw + (sg * 32 + 8 * dgl) * 4;
            col = csw + ((lane >> 5) * SGN * 32 + (lane & 31)) * 4;
            dec = sm + O_DEC + ((lane >> 5) * D + 32 * pw + (lane & 31)) * 4;
            flag = sm + O_FLAG + pw;
            row = sm + (sg * RPT * QP + f0) * ESZ;
            // feature 8 dgl + e of the wavefront's 32 goes to row rho(8 dgl + e) = 16 (dgl/2) + 8 (e/4) + 4 (dgl%2) + e%4
            // the row of feature e is R = (multiple of 8) + 4 (dgl%2) + e%4 (+ 8 (e/4)): (R/2)%4 = 2 (dgl%2) + (e/2)%2
            const uint32_t tok = rho(2 * sg), piece = tok >> 3, within = tok & 7;
#pragma unroll
            for (uint32_t x = 0; x < 2; ++x)
                kt[x] = sm + O_KT + ((32 * pw + 16 * (dgl >> 1) + 4 * (dgl & 1)) * TP + 8 * (piece ^ (2 * (dgl & 1)) ^ x) + within) * ESZ;
            // the row of column e is R = 32 pw + 8 dgl + e: (R/2)%4 = (e/2)%4
#pragma unroll
            for (uint32_t x = 0; x < 4; ++x) vt[x] = sm + O_VT + (f0 * TP + 8 * (piece ^ x) + within) * ESZ;
#pragma unroll
            for (uint32_t j = 0; j < RPT; ++j) {
                const uint32_t r = sg * RPT + j;   // the lane's 8 columns are piece dgl of quarter pw of the row
                vrow[j] = sm + O_VT + r * (D * ESZ) + 64 * (static_cast<uint32_t>(pw) ^ vswz(r)) + 16 * dgl;
                krow[j] = sm + O_KS + (kslot(r) * QP + f0) * ESZ;
            }
        }
    };

    // ------------------------------------------------------------------------------------------------------
    // Producer, gate scan of one step, in three stages with a wavefront-private LDS round trip between them.  All 16
    // token pairs of a feature live in one wavefront, so the scan over the tokens needs no workgroup barrier.  The
    // stages of step m + 1 are spread over the operand preparation of step m, which hides the round trips.
    // ------------------------------------------------------------------------------------------------------
    struct ScanOut {
        float c[2][RPT][8];   // gate sums over this thread's tokens: c[i][j] = g[0] + .. + g[j]  (times ProdAddr::unit = log2 of a decay)
        float pre[2][8];      // gate sum from the first token of the chunk to before this thread's tokens
    };
    // Gate pre-activations z -> tau log2(alpha) for alpha = sigmoid(z)^(1/tau):
    //   tau log2 alpha = min(y, 0) - log2(1 + 2^-|y|),  y = z log2 e
    // (the 1 / tau is applied where the sums are exponentiated: ProdAddr::unit).
    static __device__ __forceinline__ void activate(float (&g)[8])
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) g[e] = log2_sigmoid(g[e]);
    }
    // stage A: sums over this thread's tokens; totals of the token pair -> scan scratch.
    // `valid` = tokens of the step that exist; tokens past the end act as "no decay".
    static __device__ __forceinline__ void scan_a(const ProdAddr &pa, RawGates &r, int valid, ScanOut &o)
    {
        if (valid < S) {   // a token past the end: log-gate 0, or a pre-activation whose log-gate is exactly 0
#pragma unroll
            for (int j = 0; j < RPT; ++j)
                if (static_cast<int>(pa.sg) * RPT + j >= valid) {
                    if (pa.preact) {
                        r.g1[j].fill_huge();
                        r.g2[j].fill_huge();
                    } else {
                        r.g1[j].zero();
                        r.g2[j].zero();
                    }
                }
        }
        float g[8];
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            r.g1[j].unpack(g);
            if (pa.preact) activate(g);
#pragma unroll
            for (int e = 0; e < 8; ++e) o.c[0][j][e] = j ? o.c[0][j - 1][e] + g[e] : g[e];
            r.g2[j].unpack(g);
            if (pa.preact) activate(g);
#pragma unroll
            for (int e = 0; e < 8; ++e) o.c[1][j][e] = j ? o.c[1][j - 1][e] + g[e] : g[e];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t a = pa.tot + i * SGN * 32 * 4;
            lds_st<f32x4>(a, f32x4{o.c[i][RPT - 1][0], o.c[i][RPT - 1][1], o.c[i][RPT - 1][2], o.c[i][RPT - 1][3]});
            lds_st<f32x4>(a + 16, f32x4{o.c[i][RPT - 1][4], o.c[i][RPT - 1][5], o.c[i][RPT - 1][6], o.c[i][RPT - 1][7]});
        }
    }
    // stage B: scan of this lane's column over the 16 token pairs of the step, centred on the step: the exclusive
    // prefixes start at minus half of the step's gate sum, so that the exponents built from them span [-R/2, +R/2].
    // total: the gate sum of the column over the step (<= 0; times ProdAddr::unit = -R).
    static __device__ __forceinline__ void scan_b_read(const ProdAddr &pa, float (&t)[SGN])
    {
        wave_sync();
#pragma unroll
        for (int s2 = 0; s2 < SGN; ++s2) t[s2] = lds_ld<float>(pa.col + s2 * 32 * 4);
    }
    static __device__ __forceinline__ void scan_b(const ProdAddr &pa, const float (&t)[SGN], float &total)
    {
        float tot = (((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]))) +
                    (((t[8] + t[9]) + (t[10] + t[11])) + ((t[12] + t[13]) + (t[14] + t[15])));
        float run = -0.5f * tot;
#pragma unroll
        for (int s2 = 0; s2 < SGN; ++s2) {
            lds_st<float>(pa.col + s2 * 32 * 4, run);
            run += t[s2];
        }
        total = tot;
    }
    // bookkeeping after stage B of a step: the segment's log2 decay, and the domain check
    static __device__ __forceinline__ void note_step(const ProdAddr &pa, float total, float &seg_log2_decay, int32_t *status)
    {
        const float r = total * pa.unit;   // -R
        seg_log2_decay += r;
        if (status && !(r >= -kMaxStepLog2Decay)) *status = DSLA_STATUS_GATE_DOMAIN;
    }
    // Past this (log2) a frame change goes into the operand set as its square root and the consumers multiply by it twice:
    // the smallest normal fp32 number is 2^-126, and two neighbouring steps may move a state by up to 2^-230.
    static constexpr float kOneFactor = 120.f;
    // stage C: the exclusive prefixes of this thread's token pair
    static __device__ __forceinline__ void scan_c(const ProdAddr &pa, ScanOut &o)
    {
        wave_sync();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t a = pa.tot + i * SGN * 32 * 4;
            const f32x4 p0 = lds_ld<f32x4>(a), p1 = lds_ld<f32x4>(a + 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o.pre[i][e] = p0[e];
                o.pre[i][4 + e] = p1[e];
            }
        }
    }

    // ------------------------------------------------------------------------------------------------------
    // Producer, one call: operands of step m into operand set `set` from its inputs `r` and scan results `sc`, and,
    // interleaved, the gate scan of step m + 1 (gates `gn` -> `sn`) and the loads of later steps (`next`).
    // valid: of step m; valid_n: of step m + 1.  tot: in: gate sum of this lane's column over step m; out: over step
    // m + 1 (zero past the end of the segment).  The factor that takes the state from the middle frame of step m to
    // that of step m + 1 (to its own frame after the last step) goes into the operand set of step m.
    // ------------------------------------------------------------------------------------------------------
    template <class Loads>
    static __device__ __forceinline__ void produce(const ProdAddr &pa, uint32_t set, RawIO &r, const ScanOut &sc, int valid,
                                                   RawGates &gn, ScanOut &sn, int valid_n,
                                                   const float (&lg)[2], const uint32_t (&sgn)[2], float &tot,
                                                   float &seg_log2_decay, int32_t *status, const Loads &next)
    {
        const uint32_t so = set * SET_BYTES;
        if (valid < S) {   // ragged tail: tokens past the end act as "no key, no value"
#pragma unroll
            for (int j = 0; j < RPT; ++j)
                if (static_cast<int>(pa.sg) * RPT + j >= valid) {
                    r.k[j].zero();
                    r.v[j].zero();
                }
        }
        scan_a(pa, gn, valid_n, sn);
        next.at(0);
        next.at(1);

        Row8 kt[RPT];
        auto block = [&](int i, int j, int slot_k, int slot_q) {
            // K~ = k 2^{-c}, Q~ = gamma_i scale q 2^{c}: c = centred prefix before this thread's tokens + sum over its own
            next.at(slot_k);
            {   // row layout for the scores, token-contiguous (below) for the update
                float kf[8], kh[8];
                r.k[j].unpack(kf);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    kh[e] = kf[e] * __builtin_amdgcn_exp2f(-pa.unit * (sc.pre[i][e] + sc.c[i][j][e]));
                kt[j] = A::pack_row(kh);
                if constexpr (kTrK) A::store_row(pa.krow[j] + so + i * D * ESZ, kt[j]);
                else if (kFull) A::store_row(pa.row + so + O_KS + (j * QP + i * D) * ESZ, kt[j]);
            }
            next.at(slot_q);
            if (kFull) {
                float qf[8], qt[8];
                r.q[j].unpack(qf);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    qt[e] = qf[e] * __builtin_amdgcn_exp2f(fmaf(sc.pre[i][e] + sc.c[i][j][e], pa.unit, lg[i]));
                A::store_row(pa.row + so + O_QS + (j * QP + i * D) * ESZ, A::flip_sign(A::pack_row(qt), sgn[i]));
            }
        };
        auto kt_rows = [&](int i) {
            if constexpr (kTrK) return;   // the rows are the only copy
#pragma unroll
            for (int e = 0; e < 8; ++e)
                A::template store_tokens<RPT>(pa.kt[(e >> 1) & 1] + so + ((i * D + 8 * (e >> 2) + (e & 3)) * TP) * ESZ, kt, e);
        };

        // beta mode, tokens j: the scaled values V~ (kept for the token-contiguous copy) and the output factors
        Row8 vs[RPT];
        auto block_beta = [&](int j, int slot_a, int slot_b) {
            next.at(slot_a);
            float vf[8], vh[8], fo[8];
            r.v[j].unpack(vf);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float c = pa.unit * (sc.pre[1][e] + sc.c[1][j][e]);
                vh[e] = vf[e] * __builtin_amdgcn_exp2f(-c);
                fo[e] = __builtin_amdgcn_exp2f(c);
            }
            vs[j] = A::pack_row(vh);
            next.at(slot_b);
            if (kFull) A::store_row(pa.row + so + O_QS + (j * QP + D) * ESZ, A::pack_row(fo));
        };

        float t[SGN];
        scan_b_read(pa, t);   // the answers arrive while the first block is computed
        block(0, 0, 2, 3);
        {
            float tot_n;
            scan_b(pa, t, tot_n);
            const float change = 0.5f * pa.unit * (tot + tot_n);
            const bool twice = __builtin_amdgcn_ballot_w64(change < -kOneFactor) != 0;
            const float factor = __builtin_amdgcn_exp2f(twice ? 0.5f * change : change);
            lds_st<float>(pa.dec + so, factor);
            lds_st<float>(pa.dec + so + (O_DEC2 - O_DEC), twice ? factor : 1.f);
            if (__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0)) == 0) lds_st<uint8_t>(pa.flag + so, twice);
            note_step(pa, tot_n, seg_log2_decay, status);
            tot = tot_n;
        }
        block(0, 1, 4, 5);
        kt_rows(0);
        scan_c(pa, sn);
        if constexpr (kBeta) {
            block_beta(0, 6, 7);
            block_beta(1, 8, 9);
            if constexpr (kTrV) {
#pragma unroll
                for (int j = 0; j < RPT; ++j) A::store_row(pa.vrow[j] + so, vs[j]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) A::template store_tokens<RPT>(pa.vt[(e >> 1) & 3] + so + e * TP * ESZ, vs, e);
            }
        } else {
            block(1, 0, 6, 7);
            block(1, 1, 8, 9);
            kt_rows(1);
            if constexpr (kTrV) {   // V as loaded
#pragma unroll
                for (int j = 0; j < RPT; ++j) store_v_row(pa.vrow[j] + so, r.v[j]);
            } else {                // V transposed
#pragma unroll
                for (int e = 0; e < 8; ++e) store_v_tokens<RPT>(pa.vt[(e >> 1) & 3] + so + e * TP * ESZ, r.v, e);
            }
        }
    }

    // ------------------------------------------------------------------------------------------------------
    // Producers that load whole 128-byte lines (kLineProd: 16-bit io, ordinary step loop).  The loads and stores of the
    // step loop alone, with no arithmetic, take as long as the whole kernel, and they take 5-7 % less when a load
    // instruction fetches pieces of 128 bytes instead of 64.  So here a producer wavefront prepares ONE state, 64 features
    // of it (one line of a row), all 32 tokens: a thread has 4 tokens x 8 features.  q and k are loaded by the wavefront
    // of either state (the second request hits in L2); v is split by tokens between them.  The gate scan stays inside
    // the wavefront: sums over the thread's 4 tokens, 8 totals per feature through wavefront-private LDS, one lane per
    // feature.  The operand sets, and with them the consumers, are the ones of the row producers above.
    // ------------------------------------------------------------------------------------------------------
    static constexpr bool kLineProd = ESZ == 2 && kFull && !kExt && !kBeta && SETS == 2;
    static constexpr int FHN = D / 64;   // lines per row = producer wavefronts per state
    static constexpr int TPT = 4;        // tokens per thread
    struct LineIO {
        Raw8<TIO> q[TPT], k[TPT], v[2];
    };
    struct LineGates {
        Raw8<TG> g[TPT];
    };
    struct LineSrc {
        const TIO *q, *k, *v;   // uniform: first token of the step, this (batch, head)
        const TG *g;            // the gates of this wavefront's state
        uint32_t off[TPT];      // per lane: element offset of token 4 sq + j, features 64 fh + 8 dg ..
        uint32_t offv[2];       // the same for this wavefront's share of v: token 16 st + 2 sq + j
    };
    struct LineNext {
        LineIO &r;
        const LineSrc &rs;
        LineGates &g;
        const LineSrc &gs;
        __device__ __forceinline__ void at(int slot) const
        {
            if (slot >= 0 && slot < 4) g.g[slot].load(gs.g, gs.off[slot]);
            if (slot >= 4 && slot < 8) r.k[slot - 4].load(rs.k, rs.off[slot - 4]);
            if (slot >= 8 && slot < 12) r.q[slot - 8].load(rs.q, rs.off[slot - 8]);
            if (slot == 12) r.v[0].load(rs.v, rs.offv[0]);
            if (slot == 13) r.v[1].load(rs.v, rs.offv[1]);
        }
    };
    struct LineAddr {
        uint32_t tot;         // scan scratch [8 quads][64 features] floats: this lane's 8 features of quad sq
        uint32_t col;         // scan scratch: this lane's column (feature lane of the 64), quad 0
        uint32_t dec;         // decay factor of this lane's column
        uint32_t flag;        // how often the consumers multiply by it: of this wavefront's columns
        uint32_t qrow[TPT];   // Q~ row of token 4 sq + j, element st D + 64 fh + 8 dg
        uint32_t krow[TPT];   // K~: its row slot
        uint32_t vrow[2];     // V rows of token 16 st + 2 sq + j, columns 64 fh + 8 dg ..
        uint32_t sq, st, fh;
        bool preact;
        float unit;
        __device__ __forceinline__ LineAddr(uint32_t sm, int pw, uint32_t lane)
        {
            st = static_cast<uint32_t>(pw) / FHN;
            fh = static_cast<uint32_t>(pw) % FHN;
            sq = lane >> 3;
            const uint32_t dg = lane & 7, f0 = 64 * fh + 8 * dg;
            const uint32_t csw = sm + O_CS + pw * 4096;
            tot = csw + (sq * 64 + 8 * dg) * 4;
            col = csw + lane * 4;
            dec = sm + O_DEC + (st * D + 64 * fh + lane) * 4;
            flag = sm + O_FLAG + pw;
#pragma unroll
            for (uint32_t j = 0; j < TPT; ++j) {
                const uint32_t t = 4 * sq + j;
                qrow[j] = sm + O_QS + (t * QP + st * D + f0) * ESZ;
                krow[j] = sm + O_KS + (kslot(t) * QP + st * D + f0) * ESZ;
            }
#pragma unroll
            for (uint32_t j = 0; j < 2; ++j) {
                const uint32_t t = 16 * st + 2 * sq + j;
                vrow[j] = sm + O_VT + t * (D * ESZ) + 64 * ((f0 >> 5) ^ vswz(t)) + (f0 & 31u) * ESZ;
            }
        }
    };
    struct LineScan {
        float c[TPT][8];   // gate sums over this thread's tokens: c[j] = g[0] + .. + g[j]
        float pre[8];      // centred gate sum from the first token of the step to before this thread's tokens
    };
    static __device__ __forceinline__ void line_scan_a(const LineAddr &pa, LineGates &r, int valid, LineScan &o)
    {
        if (valid < S) {   // a token past the end: log-gate 0, or a pre-activation whose log-gate is exactly 0
#pragma unroll
            for (int j = 0; j < TPT; ++j)
                if (static_cast<int>(pa.sq) * TPT + j >= valid) {
                    if (pa.preact) r.g[j].fill_huge();
                    else r.g[j].zero();
                }
        }
        float g[8];
#pragma unroll
        for (int j = 0; j < TPT; ++j) {
            r.g[j].unpack(g);
            if (pa.preact) activate(g);
#pragma unroll
            for (int e = 0; e < 8; ++e) o.c[j][e] = j ? o.c[j - 1][e] + g[e] : g[e];
        }
        lds_st<f32x4>(pa.tot, f32x4{o.c[TPT - 1][0], o.c[TPT - 1][1], o.c[TPT - 1][2], o.c[TPT - 1][3]});
        lds_st<f32x4>(pa.tot + 16, f32x4{o.c[TPT - 1][4], o.c[TPT - 1][5], o.c[TPT - 1][6], o.c[TPT - 1][7]});
    }
    static __device__ __forceinline__ void line_scan_b_read(const LineAddr &pa, float (&t)[8])
    {
        wave_sync();
#pragma unroll
        for (int s2 = 0; s2 < 8; ++s2) t[s2] = lds_ld<float>(pa.col + s2 * 64 * 4);
    }
    // The frame of a column.  The state is kept as T with S = 2^{unit pos} T, pos the running gate sum since the frame was
    // last changed, and the exponents of a step are gate sums counted from there.  As long as pos stays within
    // kLazyFrame (log2) of zero in all 64 columns of the wavefront after the next step, the frame stays and the consumers
    // multiply nothing; otherwise it moves to the middle of the next step (after the last step: to the state itself).  A
    // move can take a column through more than fp32 holds as one factor - it is up to 115 below its frame after a step that
    // moved it, up to kLazyFrame otherwise, and the middle of the next step is up to 115 further on - so past kOneFactor
    // the consumers multiply twice by half of it (in the exponent), and no part of the history is flushed to zero.  With
    // gates of a temperature sigmoid that is once in some dozens of steps instead of 128 of the 340 vector
    // instructions of a consumer in every step; gates so strong that every step would move it behave as they always did.
    // With the 40 instructions that one exponent for both operands and the sign of the blend coefficient in q's unpacking save
    // a producer: 8 x 8192 tokens (32 heads, d = 128) 737 -> 695 us = 4.6 TB/s, 16384 tokens 279 -> 269 us, a packed batch of up
    // to 8192 tokens 665 -> 624 us.  Exponents of up to 32 cost no accuracy: they cancel between the operands, whose
    // rounding is relative (6 seeds, against 64 bits: outputs 2.73e-3 before and after; gates of very different strength
    // 2.90e-3 and 2.90e-3, states 1.65e-3 and 1.66e-3).
    static constexpr float kLazyFrame = 32.f;
    // factor, times: the state is multiplied by `factor` (per column) `times` times (uniform)
    static __device__ __forceinline__ void line_scan_b(const LineAddr &pa, const float (&t)[8], bool first_or_past, float &pos, float &factor,
                                                       uint32_t &times, float &total)
    {
        const float tot = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
        const bool move = first_or_past || __builtin_amdgcn_ballot_w64(!(fabsf((pos + tot) * pa.unit) <= kLazyFrame)) != 0;
        float run = move ? -0.5f * tot : pos;   // moved: centred on the step, as scan_b
        const float change = (pos - run) * pa.unit;
        const bool twice = __builtin_amdgcn_ballot_w64(change < -kOneFactor) != 0;
        factor = __builtin_amdgcn_exp2f(twice ? 0.5f * change : change);
        times = move ? (twice ? 2 : 1) : 0;
#pragma unroll
        for (int s2 = 0; s2 < 8; ++s2) {
            lds_st<float>(pa.col + s2 * 64 * 4, run);
            run += t[s2];
        }
        pos = run;
        total = tot;
    }
    static __device__ __forceinline__ void line_scan_c(const LineAddr &pa, LineScan &o)
    {
        wave_sync();
        const f32x4 p0 = lds_ld<f32x4>(pa.tot), p1 = lds_ld<f32x4>(pa.tot + 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o.pre[e] = p0[e] * pa.unit;
            o.pre[4 + e] = p1[e] * pa.unit;
        }
    }
    static __device__ __forceinline__ void line_note_step(const LineAddr &pa, float total, int32_t *status)
    {
        if (status && !(total * pa.unit >= -kMaxStepLog2Decay)) *status = DSLA_STATUS_GATE_DOMAIN;
    }
    // One call: operands of step m (state pa.st, 64 features) into operand set `set`, and, interleaved, the gate scan of
    // step m + 1 and the loads of later steps; as produce().  lg, sgn: of this wavefront's state.
    static __device__ __forceinline__ void line_produce(const LineAddr &pa, uint32_t set, LineIO &r, const LineScan &sc, int valid,
                                                        LineGates &gn, LineScan &sn, int valid_n, float lg, uint32_t sgn,
                                                        float &pos, int32_t *status, const LineNext &next)
    {
        const uint32_t so = set * SET_BYTES;
        if (valid < S) {   // ragged tail: tokens past the end act as "no key, no value"
#pragma unroll
            for (int j = 0; j < TPT; ++j)
                if (static_cast<int>(pa.sq) * TPT + j >= valid) r.k[j].zero();
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (static_cast<int>(16 * pa.st + 2 * pa.sq) + j >= valid) r.v[j].zero();
        }
        line_scan_a(pa, gn, valid_n, sn);
        next.at(0);
        next.at(1);
        next.at(2);
        next.at(3);
        auto block = [&](int j) {
            next.at(4 + j);
            float kf[8], kh[8], y[8];
            r.k[j].unpack(kf);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                y[e] = fmaf(sc.c[j][e], pa.unit, sc.pre[e]);
                kh[e] = kf[e] * __builtin_amdgcn_exp2f(-y[e]);
            }
            A::store_row(pa.krow[j] + so, A::pack_row(kh));
            next.at(8 + j);
            float qt[8];
#pragma unroll
            for (int w = 0; w < 4; ++w) {   // the sign of the blend coefficient enters where q is unpacked
                const uint32_t u = r.q[j].u[w];
                qt[2 * w] = __uint_as_float((u << 16) + sgn) * __builtin_amdgcn_exp2f(y[2 * w] + lg);
                qt[2 * w + 1] = __uint_as_float((u & 0xffff0000u) ^ sgn) * __builtin_amdgcn_exp2f(y[2 * w + 1] + lg);
            }
            A::store_row(pa.qrow[j] + so, A::pack_row(qt));
        };
        float t[8];
        line_scan_b_read(pa, t);   // the answers arrive while the first block is computed
        block(0);
        {
            float tot_n, factor;
            uint32_t times;
            line_scan_b(pa, t, valid_n == 0, pos, factor, times, tot_n);
            lds_st<float>(pa.dec + so, factor);
            if (threadIdx.x % 64 == 0) lds_st<uint8_t>(pa.flag + so, static_cast<uint8_t>(times));
            line_note_step(pa, tot_n, status);
        }
        block(1);
        line_scan_c(pa, sn);
        block(2);
        next.at(12);
        block(3);
        next.at(13);
#pragma unroll
        for (int j = 0; j < 2; ++j) store_v_row(pa.vrow[j] + so, r.v[j]);   // V as loaded
    }

    // ------------------------------------------------------------------------------------------------------
    // Consumer: all contractions of one step from operand set `set`.  acc[i][dt]: rows 32 dt .. of state i (Kt row
    // order), columns 32 ct ...  Register j of lane (ln, g) holds feature 32 dt + 16 (j / 8) + 8 g + j % 8.
    // Inside a chunk acc holds the state in the frame of the chunk start (see the step algebra above).
    // ------------------------------------------------------------------------------------------------------
    // Staged output rows of one step -> memory.  Consumer wavefront ct writes rows 32/CT * ct ..; a group of NC lanes
    // writes one whole row.
    static __device__ __forceinline__ void flush_rows(uint32_t sm, uint32_t parity, int ct, int lane, TIO *orow, uint32_t rs,
                                                      int valid, bool accumulate)
    {
        constexpr int RPI = 64 / NC;   // rows per instruction
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const uint32_t r = (S / CT) * ct + RPI * it + static_cast<uint32_t>(lane) / NC, c = static_cast<uint32_t>(lane) % NC;
            const uint32_t a = sm + O_ST + parity * ST_BYTES + r * (D * ESZ) + ((c ^ (r & (NC - 1))) << 4);
            u32x4 x = lds_ld<u32x4>(a);
            if (static_cast<int>(r) < valid) {
                u32x4 *dst = reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(orow) + (static_cast<size_t>(r) * rs * ESZ + c * 16));
                if (kExt && accumulate) {   // staged tiles are 16-bit: add to the eight values already there
                    const u32x4 old = *dst;
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        x[w] = ArithBf16::pack2(__uint_as_float(x[w] << 16) + __uint_as_float(old[w] << 16),
                                                __uint_as_float(x[w] & 0xffff0000u) + __uint_as_float(old[w] & 0xffff0000u));
                }
                // streaming store: the output is not read again by this call, and kept out of the caches it does not
                // delay the kernel that follows (measured: the next call's segment pre-pass 107 -> 95 us)
                __builtin_nontemporal_store(x, dst);
            }
        }
    }

    static constexpr bool kStay = ESZ == 2 && D == 128;   // the order of the MFMAs is kept: see stay()
    static __device__ __forceinline__ void consume(uint32_t sm, uint32_t set, f32x16 (&acc)[2][DT], int ct, int lane,
                                                   TIO *orow, uint32_t rs, int valid, uint32_t set_parity, bool accumulate)
    {
        const uint32_t lo = opaque(static_cast<uint32_t>(lane));
        const uint32_t ln = lo & 31, g = lo >> 5;
        const uint32_t setb = sm + set * SET_BYTES;
        // token block kb of a row: piece g + 2 kb, stored at piece position (g + 2 kb) ^ ((row / 2) % 4); all row
        // numbers used below are ln plus a multiple of 8
        const uint32_t p0 = 8 * tpiece(g, ln), p1 = 8 * tpiece(g + 2, ln);
        const uint32_t vt_r[KB] = {setb + O_VT + ((32 * ct + ln) * TP + p0) * ESZ, setb + O_VT + ((32 * ct + ln) * TP + p1) * ESZ};
        const uint32_t kt_r[KB] = {setb + O_KT + (ln * TP + p0) * ESZ, setb + O_KT + (ln * TP + p1) * ESZ};
        // transposing reads of the K~ rows (16-bit storage): lane l must end up with feature rho(l % 32) of a tile of 32
        // (the row order of the token-contiguous copy: the accumulators are fed back as fragments in it), so the lanes
        // that address piece s of 4 features point at piece (s swapped in its two bits); tokens as for V: row slots
        // 4 (l16 / 4) + g of a block of 16, and 2 slots further for the second read
        const uint32_t l16k = lo & 15, sgm = ((l16k & 1) << 1) | ((l16k >> 1) & 1);
        const uint32_t ktr_r = setb + O_KS + ((4 * (l16k >> 2) + g) * QP + 16 * ((lo >> 4) & 1) + 4 * sgm) * ESZ;
        const uint32_t dec_r = setb + O_DEC + (8 * g) * 4;
        const uint32_t moves = kLineProd ? lds_ld<uint32_t>(setb + O_FLAG) : 0u;

        // transposing reads of the V rows: the 16 lanes of a group address 4 tokens x 4 pieces of 4 columns and each
        // receives 4 tokens of ONE column; lane l ends up with column 32 ct + l % 32 and tokens 16 kb + 4 g + 0..3 (first
        // read) and 16 kb + 8 + 4 g + 0..3 (second read, 8 rows further): the order of the token-contiguous copies
        const uint32_t l16 = lo & 15, vr = 4 * g + (l16 >> 2);
        const uint32_t vs_r = setb + O_VT + vr * (D * ESZ) + 64 * (static_cast<uint32_t>(ct) ^ vswz(vr)) + 32 * ((lo >> 4) & 1) + 8 * (l16 & 3);
        Frag vf[KB];   // V fragments of this wavefront's columns: input of the output and of the update
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if constexpr (kTrV) vf[kb] = A::load_frag_tr(vs_r + 16 * kb * (D * ESZ), 8 * (D * ESZ));
            else vf[kb] = A::load_frag(vt_r[kb]);
        }

        f32x16 oacc;
        if (kFull) {
            const uint32_t qs_r = setb + O_QS + (ln * QP + 8 * g) * ESZ;
            const uint32_t ks_r = setb + O_KS + ((kTrK ? kslot(ln) : ln) * QP + 8 * g) * ESZ;
            // One pass over the 2 d_k features, 16 at a time, with the Q~ fragment shared by two products:
            //   sc[j]   = S^T[key 8(j/4) + 4g + j%4][query ln]        (Q~ K~^T, both states blended)
            //   oacc[j] = o^T[column 8(j/4) + 4g + j%4][query ln]     (carried states: the accumulators themselves
            //                                                          are the input fragments)
            f32x16 sc;
#pragma unroll
            for (int j = 0; j < 16; ++j) sc[j] = oacc[j] = 0.f;
            {
                Frag held;   // the Ks fragment of a block waits here for its Qs partner
                pipelined_steps<NST * NK, 8, A, false, kStay>(
                    [&](int s2) -> uint32_t { return ((s2 & 1) ? qs_r : ks_r) + 16 * (s2 >> 1) * ESZ; },
                    [&](int s2, const Frag &f) {
                        if ((s2 & 1) == 0) {
                            held = f;
                        } else {
                            const int kb = s2 >> 1, i = kb / (2 * DT), dt = (kb / 2) % DT, half = kb & 1;
                            A::mma(sc, held, f);
                            A::mma(oacc, A::from_acc(acc[i][dt], half), f);
                            if constexpr (kStay) {
                                stay(sc);
                                stay(oacc);
                            }
                        }
                    });
            }
            // keep key <= query; the two halves of the tile become the score fragments of the two token blocks
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint32_t key = 8 * (j >> 2) + 4 * g + (j & 3);
                sc[j] = (key <= ln) ? sc[j] : 0.f;
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) A::mma(oacc, vf[kb], A::from_acc(sc, kb));
        }
        __builtin_amdgcn_sched_barrier(0);

        // ---- add K~^T V (the output tile finishes in the matrix pipeline meanwhile) ----
        {
            constexpr int NS = KB * NST * DT;   // (token block, state, tile)
            pipelined_steps<NS, kStay ? 6 : 4, A, kTrK, kStay>(
                [&](int s2) -> uint32_t {
                    const int kb = s2 / (NST * DT), i = (s2 / DT) % NST, dt = s2 % DT;
                    if constexpr (kTrK) return ktr_r + (16 * kb * QP + i * D + 32 * dt) * ESZ;
                    else return kt_r[kb] + ((i * D + 32 * dt) * TP) * ESZ;
                },
                [&](int s2, const Frag &f) {
                    const int kb = s2 / (NST * DT), i = (s2 / DT) % NST, dt = s2 % DT;
                    A::mma(acc[i][dt], f, vf[kb]);
                    if constexpr (kStay) stay(acc[i][dt]);
                },
                2 * QP * ESZ);
            if constexpr (!kStay) {
                constexpr int RD = ESZ == 2 ? 1 : 2, MM = ESZ == 2 ? 1 : 8;
                __builtin_amdgcn_sched_group_barrier(0x100, 4 * RD, 0);
#pragma unroll
                for (int s2 = 0; s2 < NS - 4; ++s2) {
                    __builtin_amdgcn_sched_group_barrier(0x008, MM, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, RD, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 4 * MM, 0);
            }
        }

        // ---- store: lane (ln, g) holds query ln, columns 32 ct + 8 jb + 4 g .. + 3 ----
        if constexpr (kBeta && kFull) {   // the output returns from the middle frame of the columns
            const uint32_t fo_r = setb + O_QS + (ln * QP + D + 32 * ct + 4 * g) * ESZ;
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) {
                const f32x4 fo = A::load4(fo_r + 8 * jb * ESZ);
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[4 * jb + e] *= fo[e];
            }
        }
        if constexpr (kStage) {
            // piece (row ln, 16-byte piece c) lives at piece position c ^ (ln mod NC) of its row
            const uint32_t st_w = sm + O_ST + set_parity * ST_BYTES + ln * (D * ESZ) + 8 * g;
#pragma unroll
            for (int jb = 0; jb < 4; ++jb)
                A::store4(st_w + (((4 * ct + jb) ^ (ln & (NC - 1))) << 4), oacc[4 * jb], oacc[4 * jb + 1], oacc[4 * jb + 2],
                          oacc[4 * jb + 3]);
        } else if (kFull && static_cast<int>(ln) < valid) {
            TIO *op = orow + static_cast<size_t>(ln) * rs + 32 * ct + 4 * g;
#pragma unroll
            for (int jb = 0; jb < 4; ++jb) {
                float x0 = oacc[4 * jb], x1 = oacc[4 * jb + 1], x2 = oacc[4 * jb + 2], x3 = oacc[4 * jb + 3];
                if (kExt && accumulate) {
                    x0 += to_f32(op[8 * jb]);
                    x1 += to_f32(op[8 * jb + 1]);
                    x2 += to_f32(op[8 * jb + 2]);
                    x3 += to_f32(op[8 * jb + 3]);
                }
                store4_global(op + 8 * jb, x0, x1, x2, x3);
            }
        }

        // ---- the states move to the middle frame of the next step (after the last step: to their own frame), with line
        // producers those whose frame does move ----
        // (a block of its own for the register allocator: merged into the code above it costs four spilled registers)
        if constexpr (kLineProd) {
            const uint32_t m = __builtin_amdgcn_readfirstlane(moves);   // byte i FHN + f: features 64 f .. + 63 of state i
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int f = 0; f < FHN; ++f)
                    for (uint32_t times = m >> (8 * (i * FHN + f)) & 0xff; times > 0; --times) {
                        scale_tile(acc[i][2 * f], dec_r + (i * D + 64 * f) * 4);
                        scale_tile(acc[i][2 * f + 1], dec_r + (i * D + 64 * f + 32) * 4);
                    }
        } else if (opaque(1u)) {
            rescale(acc, dec_r, g, 32 * ct + ln);
            // (all tiles once more, those that need it or not: branches or loops around the tiles of one wavefront cost the
            // extended kernel at d = 128 15 to 38 spilled registers, 4 to 9 % of a call with several states)
            if (__builtin_expect((__builtin_amdgcn_readfirstlane(lds_ld<uint32_t>(setb + O_FLAG)) & (CT == 4 ? 0xffffffffu : 0xffffu)) != 0, 0))
                rescale(acc, dec_r + (O_DEC2 - O_DEC), g, 32 * ct + ln);
        }
    }

    // One 32-row tile of a state times the factors of its rows (fac: of this lane group's first row)
    static __device__ __forceinline__ void scale_tile(f32x16 &t, uint32_t fac)
    {
        f32x4 dd[4];
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) dd[jb] = lds_ld<f32x4>(fac + (16 * (jb >> 1) + 4 * (jb & 1)) * 4);
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int e = 0; e < 4; ++e) t[4 * jb + e] *= dd[jb][e];
    }
    // acc[i][dt][j] *= f[i D + feature of register j], f = 2 D floats at LDS address `fac` (+ 8 g floats for this lane);
    // beta mode: state 0 only, and every register of the lane also by the factor of the lane's column, f[D + column]
    // (`col` = the lane's column, 32 ct + ln).
    static __device__ __forceinline__ void rescale(f32x16 (&acc)[2][DT], uint32_t fac, uint32_t g, uint32_t col)
    {
        if constexpr (kBeta) {
            const float cf = lds_ld<float>(fac - 8 * g * 4 + (D + col) * 4);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int j = 0; j < 16; ++j) acc[0][dt][j] *= cf;
        }
#pragma unroll
        for (int i = 0; i < NST; ++i) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) scale_tile(acc[i][dt], fac + (i * D + 32 * dt) * 4);
        }
    }

    // The r-th longest of the B <= NT packed sequences (the earlier one where lengths are equal).  With several rounds of
    // workgroups per compute unit the last to start decide when the call ends: 37 sequences of up to 2782 tokens (32
    // heads, d = 128) take 343 us in a random order and 242 us longest first; 37 of up to 413 tokens 115 and 104 us.
    // Finding the rank costs every workgroup the loads of the lengths, four barriers and B compares per wavefront that holds a
    // sequence, before it has loaded anything: 1 to 2 us at up to 64 sequences, 3 at 256, 7 at 512 (d = 128).  order_pays()
    // has the rule.
    static __device__ int sequence_of_rank(const PrefillArgs &a, uint32_t sm, int r, int B)
    {
        typedef int i32x4 __attribute__((ext_vector_type(4)));
        const int t = threadIdx.x;
        // The length with the place below it: keys differ, so the ranks of 0 .. B - 1 are those numbers whatever the offsets
        // hold (lengths past 2^21 count as equal).
        int key = -1;
        if (t < B) {
            const int sq = a.seq ? a.seq[t] : t;
            const int len = a.cu[sq + 1] - a.cu[sq];
            key = (len < 0 ? 0 : (len < (1 << 21) ? len : 1 << 21)) * NT + (NT - 1 - t);
        }
        lds_st<int>(sm + 4 * t, key);
        __syncthreads();
        int rank = 0;
        if (t < B) {   // (wavefronts without a sequence go straight on)
            for (int u = 0; u < B; u += 4) {   // entries past the last sequence hold -1
                const i32x4 k = lds_ld<i32x4>(sm + 4 * u);
#pragma unroll
                for (int e = 0; e < 4; ++e) rank += k[e] > key ? 1 : 0;
            }
        }
        __syncthreads();
        if (t < B && rank == r) lds_st<int>(sm, t);
        __syncthreads();
        const int b = __builtin_amdgcn_readfirstlane(lds_ld<int>(sm));
        __syncthreads();
        return b;
    }

    static __device__ void run(const PrefillArgs &a, uint32_t sm)
    {
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront-uniform, kept in scalar registers

        int bidx, h;
        int64_t t0, t1;     // first token of the segment, past its last one
        size_t slot;        // workspace slot of this segment
        size_t slot_step;   // and from it to the next one's
        if (a.list_full) {
            const int it = blockIdx.x / a.H;
            if (it >= a.seg_count[kFull ? 0 : 1]) return;   // the lists are sized for the worst case
            const int4 e = (kFull ? a.list_full : a.list_pre)[it];
            bidx = e.x;
            t0 = e.y;
            t1 = e.z;
            h = blockIdx.x % a.H;
            slot_step = a.H;
            slot = static_cast<size_t>(e.w) * slot_step + h;
        } else {
            const int nseg = kFull ? a.P : a.P - 1;
            const int bh = blockIdx.x / nseg;
            const int p = blockIdx.x % nseg;
            bidx = bh / a.H;
            h = bh % a.H;
            t0 = static_cast<int64_t>(p) * a.seg_tokens;
            t1 = t0 + a.seg_tokens;
            slot_step = gridDim.x / nseg;   // B H
            slot = bh + static_cast<size_t>(p) * (kFull ? a.slot_mul : 1) * slot_step;
            if (kFull && !kExt && a.longest_first) bidx = sequence_of_rank(a, sm, bidx, static_cast<int>(slot_step) / a.H);
        }

        // this sequence: first token in the token-major tensors, length, where its states live
        const int sq = (a.cu && a.seq) ? a.seq[bidx] : bidx;
        const int64_t seq0 = a.cu ? static_cast<int64_t>(a.cu[sq]) : static_cast<int64_t>(bidx) * a.T;
        const int64_t Tb = a.cu ? static_cast<int64_t>(a.cu[sq + 1]) - seq0 : a.T;
        const size_t sbh = static_cast<size_t>(a.slot ? a.slot[bidx] : bidx) * a.H + h;
        // A shorter sequence has fewer segments: the chunk loop has nothing to do past its end, and the state
        // of a segment is only needed if another segment follows.  (Uniform exit, before any barrier.)
        if (kFull ? t0 >= Tb : t1 >= Tb) return;
        t1 = t1 < Tb ? t1 : Tb;
        const int ntok = static_cast<int>(t1 - t0);               // tokens of this segment (>= 1)
        const int nsteps = (ntok + S - 1) / S;
        const uint32_t rs = static_cast<uint32_t>(a.H) * D;       // elements between consecutive tokens
        // uniform element offset of (b, t0, h, 0); per-lane offsets are 32-bit
        const size_t seg0 = (static_cast<size_t>(seq0 + t0) * a.H + h) * D;
        const size_t sstep = static_cast<size_t>(S) * rs;
        auto valid_of = [&](int n) -> int {   // tokens of step n that exist
            const int left = ntok - n * S;
            return left >= S ? S : (left > 0 ? left : 0);
        };
        // The step loop runs in pairs (set 0, set 1), so both roles pass the same number of barriers:
        // 1 + 2 * ceil(nsteps / 2) with two sets, twice as many in the loop with one.

        if (wave < CT) {
            // =============================== consumer ===============================
            const int ct = wave;
            const int ln = lane & 31, g = lane >> 5;
            f32x16 acc[2][DT];
            const uint32_t sbase = static_cast<uint32_t>(8 * g) * D + 32 * ct + ln;   // lane part of the state offset
            // A sequence that is cut into segments starts every segment, the first one included, from the slot the
            // segment scan filled: the workgroup of the last segment overwrites the caller's states in this same
            // launch, so no workgroup of such a sequence may read them here.  A sequence of one segment reads the
            // caller's states itself (it is also the only one that writes them), unless they are zero by contract.
            const bool cut = t1 - t0 < Tb;
            // (with states that are zero by contract the first segment has nothing to read: the scan leaves its slot unwritten)
            if (kFull && (!a.zero_init || (cut && t0 > 0))) {
#pragma unroll
                for (int i = 0; i < NST; ++i) {
                    const float *src = cut ? a.ws_state + (slot * 2 + i) * D * D : (i ? a.S2 : a.S1) + sbh * D * D;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int j = 0; j < 16; ++j) acc[i][dt][j] = src[sbase + (32 * dt + 16 * (j >> 3) + (j & 7)) * D];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int j = 0; j < 16; ++j) acc[i][dt][j] = 0.f;
            }
            TIO *orow = static_cast<TIO *>(a.o) + seg0;
            const bool accum = kExt && a.accumulate;
            lds_barrier();   // operands of step 0 are ready
            if (kFull) rescale(acc, sm + O_ENT + static_cast<uint32_t>(8 * g) * 4, g, 32 * ct + ln);   // into the middle frame of step 0
            for (int n = 0; n < nsteps; n += 2) {
                if (kStage && n > 0) flush_rows(sm, 1, ct, lane, orow - sstep, rs, S, accum);
                consume(sm, 0, acc, ct, lane, orow, rs, valid_of(n), 0, accum);
                orow += sstep;
                lds_barrier();                    // step n consumed (two sets: and step n+1 ready)
                if (SETS == 1) lds_barrier();     // one set: step n+1 ready
                if (n + 1 < nsteps) {
                    if (kStage) flush_rows(sm, 0, ct, lane, orow - sstep, rs, S, accum);
                    consume(sm, SETS - 1, acc, ct, lane, orow, rs, valid_of(n + 1), 1, accum);
                    orow += sstep;
                }
                lds_barrier();
                if (SETS == 1) lds_barrier();
            }
            // the last step (every staged row has passed a barrier)
            if (kStage) flush_rows(sm, (nsteps - 1) & 1, ct, lane, orow - sstep, rs, valid_of(nsteps - 1), accum);
            // ---- write the states out ----
#pragma unroll
            for (int i = 0; i < NST; ++i) {
                float *dst = nullptr;
                if (kFull) {
                    if (t1 == Tb) dst = (i ? a.S2 : a.S1) + sbh * D * D;   // the segment with the last token
                } else {
                    // its contribution goes to the slot of the next one
                    dst = a.ws_state + ((slot + slot_step) * 2 + i) * D * D;
                }
                if (dst) {
                    const uint32_t sb = opaque(static_cast<uint32_t>(8 * g) * D + 32 * ct + ln);
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int j = 0; j < 16; ++j) dst[sb + (32 * dt + 16 * (j >> 3) + (j & 7)) * D] = acc[i][dt][j];
                }
            }
        } else {
            // =============================== producer ===============================
            const int pw = wave - CT;
            const float gm = a.gamma_per_head ? a.gamma_per_head[h] : a.gamma;
            float gsv[2] = {gm * a.scale, (1.0f - gm) * a.scale};
            if (kExt && a.explicit_w) {
                gsv[0] = (a.wa_per_head ? a.wa_per_head[h] : a.wa) * a.scale;
                gsv[1] = (a.wb_per_head ? a.wb_per_head[h] : a.wb) * a.scale;
            }
            const float lg[2] = {__builtin_amdgcn_logf(fabsf(gsv[0])), __builtin_amdgcn_logf(fabsf(gsv[1]))};
            const uint32_t sgn[2] = {gsv[0] < 0.f ? A::kSignBits : 0u, gsv[1] < 0.f ? A::kSignBits : 0u};
            if constexpr (kLineProd) {
                LineAddr pa(sm, pw, static_cast<uint32_t>(lane));
                pa.preact = a.gate_inv_tau != 0.f;
                pa.unit = pa.preact ? a.gate_inv_tau : kLog2e;
                const float lgs = pa.st ? lg[1] : lg[0];
                const uint32_t sgns = (pa.st ? gsv[1] : gsv[0]) < 0.f ? 0x80000000u : 0u;
                float pos = 0.f;   // lane l: gate sum of column (state st, feature 64 fh + l) from its frame to the end of the step scanned last
                const TIO *q0 = static_cast<const TIO *>(a.q) + seg0, *k0 = static_cast<const TIO *>(a.k) + seg0,
                          *v0 = static_cast<const TIO *>(a.v) + seg0;
                const TG *g0p = static_cast<const TG *>(pa.st ? a.g2 : a.g1) + seg0;
                const uint32_t lane_col = 64 * pa.fh + 8 * (lane & 7);
                // the lane offsets of a whole step never change; only a ragged last step clamps its rows
                uint32_t off_whole[TPT], offv_whole[2];
#pragma unroll
                for (int j = 0; j < TPT; ++j) off_whole[j] = (pa.sq * TPT + j) * rs + lane_col;
#pragma unroll
                for (int j = 0; j < 2; ++j) offv_whole[j] = (16 * pa.st + 2 * pa.sq + j) * rs + lane_col;
                auto src_of = [&](int n) -> LineSrc {   // step n, or the last step when n is past the end
                    const int m = n < nsteps ? n : nsteps - 1;
                    const size_t so = static_cast<size_t>(m) * sstep;
                    const uint32_t vm = static_cast<uint32_t>(valid_of(m));   // >= 1
                    LineSrc s;
                    s.q = q0 + so; s.k = k0 + so; s.v = v0 + so; s.g = g0p + so;
#pragma unroll
                    for (int j = 0; j < TPT; ++j) s.off[j] = off_whole[j];
#pragma unroll
                    for (int j = 0; j < 2; ++j) s.offv[j] = offv_whole[j];
                    if (vm < static_cast<uint32_t>(S)) {   // uniform
#pragma unroll
                        for (int j = 0; j < TPT; ++j) {
                            const uint32_t row = pa.sq * TPT + j;
                            s.off[j] = (row < vm ? row : vm - 1) * rs + lane_col;
                        }
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const uint32_t row = 16 * pa.st + 2 * pa.sq + j;
                            s.offv[j] = (row < vm ? row : vm - 1) * rs + lane_col;
                        }
                    }
                    return s;
                };
                auto load_gates_l = [&](LineGates &g, const LineSrc &s) {
#pragma unroll
                    for (int j = 0; j < TPT; ++j) g.g[j].load(s.g, s.off[j]);
                };
                LineIO r0, r1;
                LineGates g0, g1;
                LineScan s0, s1;
                load_gates_l(g0, src_of(0));
                load_gates_l(g1, src_of(1));
                {
                    const LineSrc s = src_of(0);
#pragma unroll
                    for (int j = 0; j < TPT; ++j) {
                        r0.k[j].load(s.k, s.off[j]);
                        r0.q[j].load(s.q, s.off[j]);
                    }
                    r0.v[0].load(s.v, s.offv[0]);
                    r0.v[1].load(s.v, s.offv[1]);
                }
                line_scan_a(pa, g0, valid_of(0), s0);
                {
                    float t[8], factor, tot;
                    uint32_t times;
                    line_scan_b_read(pa, t);
                    line_scan_b(pa, t, true, pos, factor, times, tot);
                    line_note_step(pa, tot, a.status);
                    // the caller's states enter the middle frame of step 0 (half of a step: one factor)
                    lds_st<float>(sm + O_ENT + (pa.dec - (sm + O_DEC)), factor);
                }
                line_scan_c(pa, s0);
                load_gates_l(g0, src_of(2));
                {
                    const LineSrc io = src_of(1), gs = src_of(3);
                    line_produce(pa, 0, r0, s0, valid_of(0), g1, s1, valid_of(1), lgs, sgns, pos, a.status, LineNext{r1, io, g1, gs});
                }
                lds_barrier();   // operands of step 0 are ready
                int n = 0;
                for (; n + 2 < nsteps; n += 2) {
                    {
                        const LineSrc io = src_of(n + 2), gs = src_of(n + 4);
                        line_produce(pa, 1, r1, s1, valid_of(n + 1), g0, s0, valid_of(n + 2), lgs, sgns, pos, a.status,
                                     LineNext{r0, io, g0, gs});
                    }
                    lds_barrier();
                    {
                        const LineSrc io = src_of(n + 3), gs = src_of(n + 5);
                        line_produce(pa, 0, r0, s0, valid_of(n + 2), g1, s1, valid_of(n + 3), lgs, sgns, pos, a.status,
                                     LineNext{r1, io, g1, gs});
                    }
                    lds_barrier();
                }
                // One or two steps are left and nothing is prepared past the last (a copy of its own, so that the loop above has
                // no branch around its loads): a segment of one step used to wait for two steps that do not exist.  70 tokens,
                // 32 heads, d = 128: 17.4 -> 14.9 us; 85 tokens, 16 heads, d = 64: 14.3 -> 10.9.
                if (n + 1 < nsteps) {
                    const LineSrc io = src_of(n + 2), gs = src_of(n + 4);
                    line_produce(pa, 1, r1, s1, valid_of(n + 1), g0, s0, valid_of(n + 2), lgs, sgns, pos, a.status,
                                 LineNext{r0, io, g0, gs});
                }
                lds_barrier();
                lds_barrier();
                return;
            }
            float seg_decay = 0.f;   // lane l: log2 of the segment decay of (state l / 32, feature 32 pw + l % 32)
            float tot = 0.f;         // lane l: gate sum of that column over the step whose operands come next
            ProdAddr pa(sm, pw, static_cast<uint32_t>(lane));
            pa.preact = a.gate_inv_tau != 0.f;
            pa.unit = pa.preact ? a.gate_inv_tau : kLog2e;

            // k and v of an extended launch: Hkv heads, head h reads key/value head h / (H / Hkv)
            const uint32_t rskv = kExt ? static_cast<uint32_t>(a.Hkv) * D : rs;
            const size_t seg0kv = kExt ? (static_cast<size_t>(seq0 + t0) * a.Hkv + h / (a.H / a.Hkv)) * D : seg0;
            const size_t sstepkv = static_cast<size_t>(S) * rskv;
            const TIO *q0 = static_cast<const TIO *>(a.q) + seg0, *k0 = static_cast<const TIO *>(a.k) + seg0kv,
                      *v0 = static_cast<const TIO *>(a.v) + seg0kv;
            const TG *g10 = static_cast<const TG *>(a.g1) + seg0, *g20 = static_cast<const TG *>(a.g2) + seg0;
            const uint32_t lane_col = 32 * pw + 8 * (lane & 3);
            auto src_of = [&](int n) -> StepSrc {   // step n, or the last step when n is past the end
                const int m = n < nsteps ? n : nsteps - 1;
                const size_t so = static_cast<size_t>(m) * sstep;
                const int vm = valid_of(m);   // >= 1
                StepSrc s;
                const size_t sokv = static_cast<size_t>(m) * sstepkv;
                s.q = q0 + so; s.k = k0 + sokv; s.v = v0 + sokv; s.g1 = g10 + so; s.g2 = g20 + so;
#pragma unroll
                for (int j = 0; j < RPT; ++j) {
                    uint32_t row = pa.sg * RPT + j;
                    row = row < static_cast<uint32_t>(vm) ? row : static_cast<uint32_t>(vm - 1);
                    s.off[j] = row * rs + lane_col;
                    if (kExt) s.offkv[j] = row * rskv + lane_col;
                }
                return s;
            };

            // Software pipeline over the steps, two of everything (even / odd step): while the operands of step m are
            // prepared, q, k, v of step m + 1 stream in, the gates of step m + 1 are scanned and those of step m + 3
            // stream in.
            RawIO r0, r1;
            RawGates g0, g1;
            ScanOut s0, s1;
            load_gates(g0, src_of(0));
            load_gates(g1, src_of(1));
            load_io(r0, src_of(0));
            scan_a(pa, g0, valid_of(0), s0);
            {
                float t[SGN];
                scan_b_read(pa, t);
                scan_b(pa, t, tot);
                note_step(pa, tot, seg_decay, a.status);
                // the caller's states enter the middle frame of step 0
                lds_st<float>(sm + O_ENT + (pa.dec - (sm + O_DEC)), __builtin_amdgcn_exp2f(0.5f * pa.unit * tot));
            }
            scan_c(pa, s0);
            load_gates(g0, src_of(2));
            {
                const StepSrc io = src_of(1), gs = src_of(3);
                produce(pa, 0, r0, s0, valid_of(0), g1, s1, valid_of(1), lg, sgn, tot, seg_decay, a.status,
                        NextLoads{r1, io, g1, gs});
            }
            lds_barrier();   // operands of step 0 are ready
            int n = 0;
            for (; n + 2 < nsteps; n += 2) {
                // consumers work on step n from set 0: prepare step n+1 into set 1
                if (SETS == 1) lds_barrier();     // one set: wait until step n is consumed
                {
                    const StepSrc io = src_of(n + 2), gs = src_of(n + 4);
                    produce(pa, SETS - 1, r1, s1, valid_of(n + 1), g0, s0, valid_of(n + 2), lg, sgn, tot, seg_decay,
                            a.status, NextLoads{r0, io, g0, gs});
                }
                lds_barrier();
                if (SETS == 1) lds_barrier();
                {
                    const StepSrc io = src_of(n + 3), gs = src_of(n + 5);
                    produce(pa, 0, r0, s0, valid_of(n + 2), g1, s1, valid_of(n + 3), lg, sgn, tot, seg_decay,
                            a.status, NextLoads{r1, io, g1, gs});
                }
                lds_barrier();
            }
            // the last one or two steps, as above
            if (SETS == 1) lds_barrier();
            if (n + 1 < nsteps) {
                const StepSrc io = src_of(n + 2), gs = src_of(n + 4);
                produce(pa, SETS - 1, r1, s1, valid_of(n + 1), g0, s0, valid_of(n + 2), lg, sgn, tot, seg_decay,
                        a.status, NextLoads{r0, io, g0, gs});
            }
            lds_barrier();
            if (SETS == 1) lds_barrier();
            lds_barrier();
            if (!kFull) {
                a.ws_decay[slot * 2 * D + (lane >> 5) * D + 32 * pw + (lane & 31)] = seg_decay;
            }
        }
    }
};

// Wavefronts per SIMD the register budget is set for: two, except for the fp32 step loop at d = 64, whose one
// workgroup per compute unit (LDS) is one wavefront per SIMD and whose accumulators do not fit half the register file.
template <int D, class TIO, class TG, bool kFull, bool kExt, bool kBeta = false>
__global__ __launch_bounds__(4 * D, (D == 64 && sizeof(TIO) == 4 && kFull) ? 1 : 2) void prefill_kernel(PrefillArgs a)
{
    using K = Kern<D, TIO, TG, kFull, kExt, kBeta>;
    __shared__ __attribute__((aligned(16))) char smem[K::LDS_BYTES];
    K::run(a, lds_addr_of(smem));
}

// ---------------------------------------------------------------------------------------------
// The kernels of 32-bit inputs (chunk loop, and with kFull = false the segment pre-pass): fp32 arithmetic throughout, bound by
// the fp32 matrix pipe (32 multiply-adds per clock and SIMD, a sixteenth of the bf16 rate).  The step algebra is the one above;
// what differs from the template is who does what, so that no matrix pipe idles and nothing is multiplied twice:
//  * D / 16 wavefronts, each of which prepares operands and owns 16 columns of both states (no roles), so all four SIMDs
//    multiply (with D / 32 consumers, half of them at d = 64), and D / 16 x 2 tiles of 16 x 16 leave the registers to
//    prefetch a whole step.
//  * The scores of a step are computed once: the three 16 x 16 tiles at and below the diagonal, divided over the wavefronts, meet
//    in LDS (every consumer of the template multiplies all four: a third of its matrix work).
//  * K~ and V exist once in LDS, as rows.  v_mfma_f32_16x16x4 takes one value per lane, so the token-contiguous operands of the
//    update are plain 4-byte reads (row pitches of 4 beyond a multiple of 64 floats: no conflicts); with the features of an MFMA
//    at 4 g + e the accumulators are fed back as operands and the row operands are 16-byte reads.
// Without roles, two barriers per step: operands ready; scores ready and operands read.  In between the matrix pipes are busy from
// the scores through the read-out to the update; the preparation (about a sixth of a step) is not overlapped inside a workgroup,
// at d = 64 two workgroups share a compute unit and do it for each other.
// The frame moves in every step (a frame that stays would put larger exponents, and with them larger rounding errors, into fp32
// factors): 64 multiplications, taken tile by tile in front of a tile's MFMAs, are 2 % of a step's matrix work.
// A step takes 11.5 us at d = 128 and 4.6 us at d = 64 where the template took 16.3 and 7.0 (8.1 and 2.3 of them are MFMAs at
// 2.3 GHz; the preparation is 1.0 and 1.3).  7 prompts of 1089 tokens, 32 heads, d = 128: 708 -> 450 us; 8 of 600, 32 heads, d = 64:
// 141 -> 100; one of 256, 4 heads, d = 64 (four segments): 33 -> 24.
// With roles (kRoles; d = 64, where a workgroup has its compute unit to itself: launch_f32) as many wavefronts again prepare the
// operands of step n + 1 under the MFMAs of step n, into the other of two operand sets; the scores of a step get their values after
// its one barrier, together with the read-out of the next.  A step takes 3.6 us instead of 4.6, the results are the same bits: 256
// tokens, 4 heads, whole 40.2 -> 34.0 us and in four segments 24.8 -> 24.0; 8 prompts of 600 tokens, 32 heads 109 -> 91; 50 random
// packed batches at d = 64 and 128 0.96.  At d = 128 the registers hold no second set of wavefronts and LDS no second set of operands.
// Left out: the next step prepared in registers by one wavefront of a SIMD while the other multiplies (97 spilled registers at
// d = 128: 470 instead of 362 us for 1024 tokens; at d = 64, without spills, 156 instead of 147).
// ---------------------------------------------------------------------------------------------
template <int D, class TG, bool kFull, bool kRoles>
struct F32Kern {
    using Base = Kern<D, float, TG, kFull, true, false>;   // constants of the step algebra, the order of packed sequences
    static constexpr int S = 32;                // tokens per step
    static constexpr int NW = D / 16;           // wavefronts that multiply, and that prepare: the same ones, or as many more
    static constexpr int NT = 64 * NW * (kRoles ? 2 : 1);
    static constexpr int FG = D / 32;           // wavefronts per state when preparing: wavefront w prepares state w / FG, features 32 (w % FG) ..
    static constexpr int DT = D / 16;           // 16-row tiles of a state
    static constexpr int PARTS = NW >= 6 ? 2 : 1;   // summands of a score tile: one per state, or both in one
    static constexpr int QP = 2 * D + 4, VP = D + 4, SP = S + 4;   // row pitches (floats)
    // An operand set (two with roles): Q~, K~, V; float [2D] the frame change into the step; its second factor; from the middle of the
    // step to its end; uint8 [NW] whether the second factors of a wavefront's features count.
    static constexpr uint32_t O_QS = 0, O_KS = O_QS + (kFull ? S * QP * 4 : 0), O_V = O_KS + S * QP * 4, O_DEC = O_V + S * VP * 4;
    static constexpr uint32_t O_DEC2 = O_DEC + 2 * D * 4, O_END = O_DEC2 + 2 * D * 4, O_FLAG = O_END + 2 * D * 4;
    static constexpr uint32_t SET_BYTES = O_FLAG + 16, SC_BYTES = kFull ? PARTS * S * SP * 4 : 0;
    static constexpr uint32_t O_SC = SET_BYTES * (kRoles ? 2 : 1);                  // scores of a step
    static constexpr uint32_t O_CS = O_SC + SC_BYTES * (kRoles ? 2 : 1);            // per wavefront: float [16][32] scan scratch
    static constexpr uint32_t LDS_BYTES = O_CS + NW * 2048;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");

    struct Raw {   // inputs of one step as loaded: 2 tokens x 8 features of q, k and one state's gates, 1 token x 8 columns of v
        Raw8<float> q[2], k[2], v;
        Raw8<TG> g[2];
    };

    static __device__ __forceinline__ void run(const PrefillArgs &a, uint32_t sm)
    {
        const int lane = threadIdx.x & 63, wave_id = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
        const int wave = wave_id % NW;   // among those of its role
        const bool prepares = wave_id >= NW;

        // ---- the work item: as Kern::run ----
        int bidx, h;
        int64_t t0, t1;
        size_t slot, slot_step;
        if (a.list_full) {
            const int it = blockIdx.x / a.H;
            if (it >= a.seg_count[kFull ? 0 : 1]) return;
            const int4 e = (kFull ? a.list_full : a.list_pre)[it];
            bidx = e.x;
            t0 = e.y;
            t1 = e.z;
            h = blockIdx.x % a.H;
            slot_step = a.H;
            slot = static_cast<size_t>(e.w) * slot_step + h;
        } else {
            const int nseg = kFull ? a.P : a.P - 1;
            const int bh = blockIdx.x / nseg;
            const int p = blockIdx.x % nseg;
            bidx = bh / a.H;
            h = bh % a.H;
            t0 = static_cast<int64_t>(p) * a.seg_tokens;
            t1 = t0 + a.seg_tokens;
            slot_step = gridDim.x / nseg;
            slot = bh + static_cast<size_t>(p) * (kFull ? a.slot_mul : 1) * slot_step;
            if (kFull && a.longest_first) bidx = Base::sequence_of_rank(a, sm, bidx, static_cast<int>(slot_step) / a.H);
        }
        const int sq = (a.cu && a.seq) ? a.seq[bidx] : bidx;
        const int64_t seq0 = a.cu ? static_cast<int64_t>(a.cu[sq]) : static_cast<int64_t>(bidx) * a.T;
        const int64_t Tb = a.cu ? static_cast<int64_t>(a.cu[sq + 1]) - seq0 : a.T;
        const size_t sbh = static_cast<size_t>(a.slot ? a.slot[bidx] : bidx) * a.H + h;
        if (kFull ? t0 >= Tb : t1 >= Tb) return;   // (uniform, before any barrier)
        t1 = t1 < Tb ? t1 : Tb;
        const int ntok = static_cast<int>(t1 - t0), nsteps = (ntok + S - 1) / S;
        const uint32_t rs = static_cast<uint32_t>(a.H) * D, rskv = static_cast<uint32_t>(a.Hkv) * D;   // elements between tokens
        const size_t seg0 = (static_cast<size_t>(seq0 + t0) * a.H + h) * D;
        const size_t seg0kv = (static_cast<size_t>(seq0 + t0) * a.Hkv + h / (a.H / a.Hkv)) * D;

        // ---- preparing: lane (sg, dgl) has tokens 2 sg, 2 sg + 1 and features 32 pw + 8 dgl .. of state st; of v token 16 st + sg ----
        const uint32_t st = static_cast<uint32_t>(wave) / FG, pw = static_cast<uint32_t>(wave) % FG;
        const uint32_t sg = static_cast<uint32_t>(lane) >> 2, f0 = 32 * pw + 8 * (lane & 3u);
        const uint32_t fcol = static_cast<uint32_t>(lane) & 31u, hh = static_cast<uint32_t>(lane) >> 5;   // scan: feature, half of the token pairs
        const uint32_t cs = sm + O_CS + wave * 2048, cs_own = cs + (sg * 32 + 8 * (lane & 3u)) * 4, cs_col = cs + (8 * hh * 32 + fcol) * 4;
        const uint32_t decl = (st * D + 32 * pw + fcol) * 4;
        const bool preact = a.gate_inv_tau != 0.f;
        const float unit = preact ? a.gate_inv_tau : kLog2e;   // gate sums times this = log2 of a decay
        float gs;
        if (a.explicit_w) {
            const float *per_head = st ? a.wb_per_head : a.wa_per_head;
            gs = (per_head ? per_head[h] : (st ? a.wb : a.wa)) * a.scale;
        } else {
            const float gm = a.gamma_per_head ? a.gamma_per_head[h] : a.gamma;
            gs = (st ? 1.0f - gm : gm) * a.scale;
        }
        const float lg = __builtin_amdgcn_logf(fabsf(gs));
        const uint32_t sgn = gs < 0.f ? 0x80000000u : 0u;
        const float *q0 = static_cast<const float *>(a.q) + seg0, *k0 = static_cast<const float *>(a.k) + seg0kv,
                    *v0 = static_cast<const float *>(a.v) + seg0kv;
        const TG *gate0 = static_cast<const TG *>(st ? a.g2 : a.g1) + seg0;
        auto valid_of = [&](int n) -> int {
            const int left = ntok - n * S;
            return left >= S ? S : left;
        };
        auto load = [&](Raw &x, int n) {   // step n < nsteps; a token past the end re-reads the last one
            const size_t so = static_cast<size_t>(n) * S * rs, sokv = static_cast<size_t>(n) * S * rskv;
            const uint32_t last = static_cast<uint32_t>(valid_of(n)) - 1;
            auto row = [&](uint32_t t) { return t < last ? t : last; };
#pragma unroll
            for (uint32_t j = 0; j < 2; ++j) x.g[j].load(gate0 + so, row(2 * sg + j) * rs + f0);
#pragma unroll
            for (uint32_t j = 0; j < 2; ++j) {
                x.k[j].load(k0 + sokv, row(2 * sg + j) * rskv + f0);
                if (kFull) x.q[j].load(q0 + so, row(2 * sg + j) * rs + f0);
            }
            x.v.load(v0 + sokv, row(16 * st + sg) * rskv + f0);
        };
        float tot = 0.f, seg_decay = 0.f;   // of this lane's scan column: gate sum of the step prepared last, log2 decay of the segment
        auto prepare = [&](Raw &x, int valid, uint32_t set) {   // set: of the operands (bytes)
            float c[2][8];   // gate sums over this thread's tokens
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                x.g[j].unpack(c[j]);
                if (preact) Base::activate(c[j]);
                if (static_cast<int>(2 * sg) + j >= valid) {   // past the end: no decay, no key
#pragma unroll
                    for (int e = 0; e < 8; ++e) c[j][e] = 0.f;
                    x.k[j].zero();
                }
            }
            if (static_cast<int>(16 * st + sg) >= valid) x.v.zero();
#pragma unroll
            for (int e = 0; e < 8; ++e) c[1][e] += c[0][e];
            lds_st<f32x4>(cs_own, f32x4{c[1][0], c[1][1], c[1][2], c[1][3]});
            lds_st<f32x4>(cs_own + 16, f32x4{c[1][4], c[1][5], c[1][6], c[1][7]});
            const uint32_t va = sm + set + O_V + ((16 * st + sg) * VP + f0) * 4;
            lds_st<f32x4>(va, x.v.a);
            lds_st<f32x4>(va + 16, x.v.b);
            Base::wave_sync();
            {   // the scan over the 16 token pairs of a feature, 8 to a lane; centred on the step (see the step algebra)
                float t[8];
#pragma unroll
                for (int s2 = 0; s2 < 8; ++s2) t[s2] = lds_ld<float>(cs_col + s2 * 128);
                const float mine = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7])), other = __shfl_xor(mine, 32);
                const float sum = mine + other;
                float run = -0.5f * sum + (hh ? other : 0.f);
#pragma unroll
                for (int s2 = 0; s2 < 8; ++s2) {
                    lds_st<float>(cs_col + s2 * 128, run);
                    run += t[s2];
                }
                // from the middle of the step before (or the state itself) to the middle of this one; past one factor as two equal ones
                const float change = 0.5f * unit * (tot + sum);
                const bool twice = __builtin_amdgcn_ballot_w64(change < -Base::kOneFactor) != 0;
                const float factor = __builtin_amdgcn_exp2f(twice ? 0.5f * change : change);
                lds_st<float>(sm + set + O_DEC + decl, factor);   // (both lanes of a feature write the same)
                lds_st<float>(sm + set + O_DEC2 + decl, twice ? factor : 1.f);
                lds_st<float>(sm + set + O_END + decl, __builtin_amdgcn_exp2f(0.5f * unit * sum));
                if (lane == 0) lds_st<uint8_t>(sm + set + O_FLAG + wave, twice);
                tot = sum;
                const float r = sum * unit;
                seg_decay += r;
                if (a.status && !(r >= -kMaxStepLog2Decay)) *a.status = DSLA_STATUS_GATE_DOMAIN;
            }
            Base::wave_sync();
            const f32x4 p0 = lds_ld<f32x4>(cs_own), p1 = lds_ld<f32x4>(cs_own + 16);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float kf[8], qf[8];
                x.k[j].unpack(kf);
                if (kFull) x.q[j].unpack(qf);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float y = (e < 4 ? p0[e & 3] : p1[e & 3]) + c[j][e];
                    kf[e] *= __builtin_amdgcn_exp2f(-unit * y);
                    if (kFull) qf[e] = __uint_as_float(__float_as_uint(qf[e]) ^ sgn) * __builtin_amdgcn_exp2f(fmaf(y, unit, lg));
                }
                const uint32_t at = set + ((2 * sg + j) * QP + st * D + f0) * 4;
                lds_st<f32x4>(sm + O_KS + at, f32x4{kf[0], kf[1], kf[2], kf[3]});
                lds_st<f32x4>(sm + O_KS + at + 16, f32x4{kf[4], kf[5], kf[6], kf[7]});
                if (kFull) {
                    lds_st<f32x4>(sm + O_QS + at, f32x4{qf[0], qf[1], qf[2], qf[3]});
                    lds_st<f32x4>(sm + O_QS + at + 16, f32x4{qf[4], qf[5], qf[6], qf[7]});
                }
            }
        };

        if (kRoles && prepares) {
            Raw x;
            load(x, 0);
            prepare(x, valid_of(0), 0);
            if (nsteps > 1) load(x, 1);
            lds_barrier();   // the operands of step 0 are ready
            for (int n = 0; n < nsteps; ++n) {
                if (n + 1 < nsteps) {
                    prepare(x, valid_of(n + 1), ((n + 1) & 1) * SET_BYTES);
                    if (n + 2 < nsteps) load(x, n + 2);
                }
                lds_barrier();   // those of step n + 1 are, and step n has been read
            }
            if (!kFull && lane < 32) a.ws_decay[slot * 2 * D + st * D + 32 * pw + fcol] = seg_decay;
            return;
        }

        // ---- multiplying: lane (r, g); acc[i][dt][e] = T^i[16 dt + 4 g + e][16 wave + r] ----
        const uint32_t r = lane & 15, g = static_cast<uint32_t>(lane) >> 4;
        f32x4 acc[2][DT];
        const bool cut = t1 - t0 < Tb;   // (which states a segment starts from: see Kern::run)
        const uint32_t sbase = 4 * g * D + 16 * wave + r;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (kFull && (!a.zero_init || (cut && t0 > 0))) {
                const float *src = cut ? a.ws_state + (slot * 2 + i) * D * D : (i ? a.S2 : a.S1) + sbh * D * D;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][dt][e] = src[sbase + (16 * dt + e) * D];
            } else {
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) acc[i][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        auto scale = [&](uint32_t factors, int i, int dt) {
            const f32x4 f = lds_ld<f32x4>(factors + (i * D + 16 * dt + 4 * g) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][dt][e] *= f[e];
        };
        auto rescale = [&](uint32_t factors) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) scale(factors, i, dt);
        };
        auto mma = [](f32x4 &c, float x, float y) { c = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0); };

        float vf[2][4];   // V[16 kt + 4 g + e][16 wave + r]: operand of the output and of the update
        f32x4 oacc[2];    // o[16 qt + 4 g + e][16 wave + r]
        // scores, read-out and update of step n from its operand set; the scores go to LDS at sm + O_SC + sc_at
        auto product = [&](int n, uint32_t set, uint32_t sc_at) {
            const uint32_t sb = sm + set;
            const uint32_t qrow = sb + O_QS + (r * QP + 4 * g) * 4, krow = sb + O_KS + (r * QP + 4 * g) * 4;   // row r, features 4 g ..
            const uint32_t kcol = sb + O_KS + (4 * g * QP + r) * 4;                    // K~[4 g][r]
            const uint32_t vcol = sb + O_V + (4 * g * VP + 16 * wave + r) * 4;         // V[4 g][16 wave + r]
            auto move = [&](int i, int dt) { scale(sb + O_DEC, i, dt); };   // into the middle frame of the step, tile by tile under the MFMAs
            bool again = false;
#pragma unroll
            for (int w = 0; w < NW; w += 4) again |= __builtin_amdgcn_readfirstlane(lds_ld<uint32_t>(sb + O_FLAG + w)) != 0;
            if (__builtin_expect(again, 0)) rescale(sb + O_DEC2);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int e = 0; e < 4; ++e) vf[kt][e] = lds_ld<float>(vcol + (16 * kt + e) * VP * 4);

            if constexpr (kFull) {
                // a score tile (queries 16 qt .., keys 16 kt ..; (0, 0), (1, 0), (1, 1)) or its share of one state
                if (wave < 3 * PARTS) {
                    const int tile = wave % 3, part = wave / 3, qt = tile > 0, kt = tile > 1;
                    constexpr int NB = 2 * D / PARTS / 16;   // blocks of 16 features
                    const uint32_t qa = qrow + (16 * qt * QP + part * D) * 4, ka = krow + (16 * kt * QP + part * D) * 4;
                    f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const f32x4 qv = lds_ld<f32x4>(qa + b * 64), kv = lds_ld<f32x4>(ka + b * 64);
#pragma unroll
                        for (int e = 0; e < 4; ++e) mma(sc[e & 1], qv[e], kv[e]);
                    }
                    const uint32_t out = sm + O_SC + sc_at + ((part * S + 16 * qt + 4 * g) * SP + 16 * kt + r) * 4;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        lds_st<float>(out + e * SP * 4, 16 * kt + r <= 16 * qt + 4 * g + e ? sc[0][e] + sc[1][e] : 0.f);
                }
#pragma unroll
                for (int qt = 0; qt < 2; ++qt) oacc[qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) {
                        move(i, dt);
                        const f32x4 qa = lds_ld<f32x4>(qrow + (i * D + 16 * dt) * 4), qb = lds_ld<f32x4>(qrow + (16 * QP + i * D + 16 * dt) * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            mma(oacc[0], qa[e], acc[i][dt][e]);
                            mma(oacc[1], qb[e], acc[i][dt][e]);
                        }
                    }
            }
            // T += K~^T V
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (!kFull && kt == 0 && e == 0) move(i, dt);
                            mma(acc[i][dt], lds_ld<float>(kcol + ((16 * kt + e) * QP + i * D + 16 * dt) * 4), vf[kt][e]);
                        }
            if (n + 1 == nsteps) rescale(sb + O_END);
        };
        // the scores' share of the output of step n, and its rows
        auto output = [&](int n, uint32_t sc_at) {
            if constexpr (kFull) {
                const uint32_t sa = sm + O_SC + sc_at + (r * SP + 4 * g) * 4;
                auto weights = [&](int qt, int kt) {
                    f32x4 w = lds_ld<f32x4>(sa + (16 * qt * SP + 16 * kt) * 4);
                    if (PARTS == 2) {
                        const f32x4 w2 = lds_ld<f32x4>(sa + ((S + 16 * qt) * SP + 16 * kt) * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] += w2[e];
                    }
                    return w;
                };
                const f32x4 w00 = weights(0, 0), w10 = weights(1, 0), w11 = weights(1, 1);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    mma(oacc[0], w00[e], vf[0][e]);
                    mma(oacc[1], w10[e], vf[0][e]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) mma(oacc[1], w11[e], vf[1][e]);
                const int valid = valid_of(n);
                float *orow = static_cast<float *>(a.o) + seg0 + static_cast<size_t>(n) * S * rs + 16 * wave + r;
                if (a.accumulate) {
#pragma unroll
                    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (static_cast<int>(16 * qt + 4 * g + e) < valid) oacc[qt][e] += orow[(16 * qt + 4 * g + e) * rs];
                }
#pragma unroll
                for (int qt = 0; qt < 2; ++qt)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (static_cast<int>(16 * qt + 4 * g + e) < valid) orow[(16 * qt + 4 * g + e) * rs] = oacc[qt][e];
            }
        };
        if constexpr (kRoles) {
            lds_barrier();   // the operands of step 0 are ready
            for (int n = 0; n < nsteps; ++n) {
                if (n > 0) output(n - 1, ((n - 1) & 1) * SC_BYTES);
                product(n, (n & 1) * SET_BYTES, (n & 1) * SC_BYTES);
                lds_barrier();   // the scores of step n and the operands of step n + 1 are there
            }
            output(nsteps - 1, ((nsteps - 1) & 1) * SC_BYTES);
        } else {
            Raw x;
            load(x, 0);
            for (int n = 0; n < nsteps; ++n) {
                prepare(x, valid_of(n), 0);
                if (n + 1 < nsteps) load(x, n + 1);
                lds_barrier();   // the operands of step n are ready
                product(n, 0, 0);
                lds_barrier();   // the scores are there; everybody has read the operands of step n
                output(n, 0);
            }
        }
        // ---- the states: of the segment with the last token to the caller, a segment's contribution to slot p + 1 ----
        if (!kFull || t1 == Tb) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float *dst = kFull ? (i ? a.S2 : a.S1) + sbh * D * D : a.ws_state + ((slot + slot_step) * 2 + i) * D * D;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) dst[sbase + (16 * dt + e) * D] = acc[i][dt][e];
            }
        }
        if (!kFull && !kRoles && lane < 32) a.ws_decay[slot * 2 * D + st * D + 32 * pw + fcol] = seg_decay;
    }
};
template <int D, class TG, bool kFull, bool kRoles>
__global__ __launch_bounds__((F32Kern<D, TG, kFull, kRoles>::NT), 2) void prefill_f32_kernel(PrefillArgs a)
{
    using K = F32Kern<D, TG, kFull, kRoles>;
    __shared__ __attribute__((aligned(16))) char smem[K::LDS_BYTES];
    K::run(a, lds_addr_of(smem));
}

// ---------------------------------------------------------------------------------------------
// Segment pre-pass of its own design for the common case: 16-bit io and gates, d = 128, two states.
//
// The state contribution of a segment of N tokens is U^i = sum_t diag(prod_{s > t} alpha^i_s) k_t^T v_t (Section 4.1,
// the state update unrolled to the end of the segment).  Walking the segment BACKWARDS, 32 tokens at a time, the
// exponent of every factor is a running suffix sum of log-gates: never positive, so nothing is centred and the
// accumulated state is never rescaled:
//     K~^i_t = k_t 2^{E^i_t},  E^i_t = sum_{s > t} log2 alpha^i_s  (<= 0)        U^i += (K~^i)^T V      per step.
// Inputs reach LDS as whole rows through loads that write LDS directly (no registers, 2 steps ahead of their use:
// 64 KB per workgroup in flight).  The suffix sums over the 32 tokens of a step are a product of a constant 0/1
// matrix with the tile of log-gates: the matrix unit evaluates them, exactly, and hands every lane one feature and 16
// tokens of it; a transposing LDS read delivers the keys in the same arrangement, and what is left for the vector unit
// is one fused multiply-add, one exponential, one multiply and half a pack per (token, feature, state): a third of
// what the producer wavefronts of the step-loop template spend on the same operands.
//
// All 8 wavefronts do both jobs: wavefront w prepares state w / 4, features 32 (w % 4) .. + 31, and multiplies
// state w / 4, columns 32 (w % 4) .. + 31 (64 accumulator registers).  One barrier per step: in interval n every
// wavefront prepares K~ of step n into one of two K~ buffers and then multiplies step n - 1, so the vector and the
// matrix work of neighbouring steps overlap across the wavefronts of a SIMD.
// LDS: 3 slots of (k, g1, g2) rows + 4 slots of v rows + 2 K~ buffers = 72 + 32 + 32 KB.  All rows as loaded, the
// 64-byte quarter q of row r at quarter position q ^ (r % 4) (every tensor is read transposed); K~ as in the
// step-loop template: [i D + feature][rho(token)], piece c of row R at c ^ ((R / 2) % 4).
// ---------------------------------------------------------------------------------------------
struct SegFast {
    static constexpr int D = 128, S = 32;
    static constexpr int NWAVE = 8, NT = 64 * NWAVE;
    static constexpr int LEAD = 2;                                     // steps between a load and its use
    static constexpr int KG_SLOTS = LEAD + 1, V_SLOTS = LEAD + 2;      // v lives one interval longer (it is multiplied one later)
    static constexpr uint32_t ROWB = D * 2, TEN = S * ROWB;            // a row, a tensor of one step (bytes)
    static constexpr uint32_t KG_BYTES = 3 * TEN;
    static constexpr uint32_t O_KG = 0, O_V = O_KG + KG_SLOTS * KG_BYTES, O_KT = O_V + V_SLOTS * TEN;
    static constexpr uint32_t KT_BYTES = 2 * D * S * 2;
    static constexpr uint32_t LDS_BYTES = O_KT + 2 * KT_BYTES;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS budget");
};

// 16 bytes per lane from `base` (wavefront-uniform) + `voff` (per lane) into LDS at `lds` (uniform) + 16 * lane.
// The compiler does not know these loads: whoever reads the bytes waits with wait_loads<>() first.
// (M0 holds the LDS address; the compiler reserves that register for instructions of this kind and is told that it changes.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds16(uint32_t lds, uint32_t voff, const char *base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_loads_and_barrier()   // at most N of this wavefront's loads still in flight; then the workgroup meets
{
    static_assert(N == 0 || N == 4, "one step of loads is 4 instructions per wavefront");
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (N == 4) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ const char *uniform_ptr(const void *p)   // the same pointer, held in scalar registers
{
    const uint64_t x = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x)));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32)));
    return reinterpret_cast<const char *>((static_cast<uint64_t>(hi) << 32) | lo);
}
__global__ __launch_bounds__(SegFast::NT, 2) void segment_state_fast_kernel(PrefillArgs a)
{
    using F = SegFast;
    using A = ArithBf16;
    constexpr int D = F::D, S = F::S;
    __shared__ __attribute__((aligned(1024))) char smem[F::LDS_BYTES];
    const uint32_t sm = lds_addr_of(smem);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));

    // the work item: as Kern::run with kFull = false
    int bidx, h;
    int64_t t0, t1;
    size_t slot, slot_step;
    if (a.list_full) {
        const int it = blockIdx.x / a.H;
        if (it >= a.seg_count[1]) return;
        const int4 e = a.list_pre[it];
        bidx = e.x;
        t0 = e.y;
        t1 = e.z;
        h = blockIdx.x % a.H;
        slot_step = a.H;
        slot = static_cast<size_t>(e.w) * slot_step + h;
    } else {
        const int nseg = a.P - 1;
        const int bh = blockIdx.x / nseg;
        const int p = blockIdx.x % nseg;
        bidx = bh / a.H;
        h = bh % a.H;
        t0 = static_cast<int64_t>(p) * a.seg_tokens;
        t1 = t0 + a.seg_tokens;
        slot_step = gridDim.x / nseg;
        slot = bh + p * slot_step;
    }
    const int sq = (a.cu && a.seq) ? a.seq[bidx] : bidx;
    const int64_t seq0 = a.cu ? static_cast<int64_t>(a.cu[sq]) : static_cast<int64_t>(bidx) * a.T;
    const int64_t Tb = a.cu ? static_cast<int64_t>(a.cu[sq + 1]) - seq0 : a.T;
    if (t1 >= Tb) return;   // no segment follows: nobody needs this one's contribution (uniform exit)
    // what is followed by another segment is whole: a multiple of a step
    const int nsteps = static_cast<int>(t1 - t0) / S;
    const uint32_t rs2 = static_cast<uint32_t>(a.H) * D * 2;   // bytes between consecutive tokens
    const size_t seg0 = (static_cast<size_t>(seq0 + t0) * a.H + h) * D * 2;
    const size_t step_bytes = static_cast<size_t>(S) * rs2;
    // k and v may have fewer heads (extended launches): head h reads key/value head h / (H / Hkv)
    const uint32_t rs2kv = static_cast<uint32_t>(a.Hkv) * D * 2;
    const size_t seg0kv = (static_cast<size_t>(seq0 + t0) * a.Hkv + h / (a.H / a.Hkv)) * D * 2;
    const size_t step_bytes_kv = static_cast<size_t>(S) * rs2kv;
    const char *pk = uniform_ptr(static_cast<const char *>(a.k) + seg0kv), *pv = uniform_ptr(static_cast<const char *>(a.v) + seg0kv),
               *pg1 = uniform_ptr(static_cast<const char *>(a.g1) + seg0), *pg2 = uniform_ptr(static_cast<const char *>(a.g2) + seg0);

    // ---- loading: wavefront w brings rows 4 w .. 4 w + 3 of every tensor of a step, lane l piece position l % 16 of row l / 16 ----
    const uint32_t drow = 4 * wave + (lane >> 4), dpos = lane & 15;
    const uint32_t dpiece = ((((dpos >> 2) ^ (drow & 3u)) << 2) | (dpos & 3u)) << 4;
    const uint32_t voff = drow * rs2 + dpiece, voff_kv = drow * rs2kv + dpiece;
    auto issue = [&](uint32_t kg_slot, uint32_t v_slot, int n) {   // step n of the walk = step nsteps - 1 - n of the segment
        const size_t off = static_cast<size_t>(nsteps - 1 - n) * step_bytes, off_kv = static_cast<size_t>(nsteps - 1 - n) * step_bytes_kv;
        const uint32_t kgb = sm + F::O_KG + kg_slot * F::KG_BYTES + wave * 1024;
        load_to_lds16(kgb, voff_kv, pk + off_kv);
        load_to_lds16(kgb + F::TEN, voff, pg1 + off);
        load_to_lds16(kgb + 2 * F::TEN, voff, pg2 + off);
        load_to_lds16(sm + F::O_V + v_slot * F::TEN + wave * 1024, voff_kv, pv + off_kv);
    };

    // Both jobs of wavefront w concern state st = w / 4 and the 32-tile ct = w % 4: features 32 ct .. of the keys and gates
    // when preparing, columns 32 ct .. of the values when multiplying.  A transposing read of staged rows hands lane
    // (ln, g) column 32 ct + ln and, for token block kb, the 8 tokens tau(kb, g, e) = 16 kb + 8 (e / 4) + 4 g + e % 4 --
    // an MFMA input fragment whose contraction index runs over the tokens in that order.
    const uint32_t st = wave >> 2, ct = wave & 3, ln = lane & 31, g = lane >> 5, l16 = lane & 15, vr = 4 * g + (l16 >> 2);
    const uint32_t tr_r = vr * F::ROWB + 64 * (ct ^ (vr & 3u)) + 32 * ((lane >> 4) & 1u) + 8 * (l16 & 3u);   // inside a staged tensor
    auto rows_frag = [&](uint32_t tensor, int kb) { return A::load_frag_tr(tensor + tr_r + 16 * kb * F::ROWB, 8 * F::ROWB); };
    // K~ rows: lane (ln, g) writes (preparing) and reads (multiplying) piece g + 2 kb of row st D + 32 tile + ln
    const uint32_t kt_r = sm + F::O_KT + (st * D + ln) * 64;
    const uint32_t kt_p[2] = {(g ^ ((ln >> 1) & 3u)) << 4, ((g + 2) ^ ((ln >> 1) & 3u)) << 4};

    // ---- preparing ----
    // The exponents of a step are suffix sums of its log-gates over the tokens: E[t][f] = sum_{t' > t} g[t'][f], a product
    // of a constant 0/1 matrix with the gate tile, which the matrix unit evaluates exactly (bf16 gates times 0 or 1, fp32
    // sums): tri[kb] is row ln of that matrix as the fragment whose contraction index runs over tau(kb, g, .).  The result
    // tile hands lane (ln, g) feature 32 ct + ln and, in register j, token 8 (j / 4) + 4 g + j % 4 = tau(j / 8, g, j % 8): the
    // order in which a transposing read delivers the keys, and 8 consecutive positions of a K~ row.
    A::Frag tri[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        u32x4 u;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t t_lo = 16 * kb + 8 * ((2 * w) >> 2) + 4 * g + ((2 * w) & 3), t_hi = t_lo + 1;
            u[w] = (t_lo > ln ? 0x3f80u : 0u) | (t_hi > ln ? 0x3f800000u : 0u);   // bf16 1.0 = 0x3f80
        }
        tri[kb].v = __builtin_bit_cast(bf16x8, u);
    }
    const bool preact = a.gate_inv_tau != 0.f;
    const float unit = preact ? a.gate_inv_tau : kLog2e;   // gate sums times this = log2 of a decay
    float carry = 0.f;   // gate sum over all later steps of the segment, feature 32 ct + ln of state st (the same in both lane groups)

    auto prepare = [&](uint32_t kg_slot, uint32_t kt_buf) {
        const uint32_t kbase = sm + F::O_KG + kg_slot * F::KG_BYTES, gbase = kbase + (1 + st) * F::TEN;
        A::Frag gf[2], kf[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) gf[kb] = rows_frag(gbase, kb);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) kf[kb] = rows_frag(kbase, kb);
        f32x16 E;
#pragma unroll
        for (int j = 0; j < 16; ++j) E[j] = 0.f;
        float g_first;   // the gate of token tau(0, g, 0) = 4 g
        if (!preact) {
            A::mma(E, tri[0], gf[0]);
            A::mma(E, tri[1], gf[1]);
            g_first = __uint_as_float(__builtin_bit_cast(u32x4, gf[0].v)[0] << 16);
        } else {
            // pre-activations z -> tau log2 alpha (as Kern::activate); the result is not a bf16 number: it enters the
            // matrix unit as the sum of two (hi + lo: 16 mantissa bits)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                const u32x4 zw = __builtin_bit_cast(u32x4, gf[kb].v);
                u32x4 hi, lo;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    float x[2] = {__uint_as_float(zw[w] << 16), __uint_as_float(zw[w] & 0xffff0000u)};
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float y = x[e] * kLog2e;
                        x[e] = fminf(y, 0.f) - __builtin_amdgcn_logf(1.0f + __builtin_amdgcn_exp2f(-__builtin_fabsf(y)));
                    }
                    if (kb == 0 && w == 0) g_first = x[0];
                    hi[w] = A::pack2(x[0], x[1]);
                    lo[w] = A::pack2(x[0] - __uint_as_float(hi[w] << 16), x[1] - __uint_as_float(hi[w] & 0xffff0000u));
                }
                A::Frag fh, fl;
                fh.v = __builtin_bit_cast(bf16x8, hi);
                fl.v = __builtin_bit_cast(bf16x8, lo);
                A::mma(E, tri[kb], fh);
                A::mma(E, tri[kb], fl);
            }
        }
        // gate sum of the whole step = E[token 0] + g[token 0]: lane group 0 has it, group 1 fetches it
        const float tot = __int_as_float(__builtin_amdgcn_ds_bpermute(static_cast<int>(ln << 2), __float_as_int(E[0] + g_first)));
        const float cu = carry * unit;
        carry += tot;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const u32x4 kw = __builtin_bit_cast(u32x4, kf[kb].v);
            u32x4 out;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float k0 = __uint_as_float(kw[w] << 16), k1 = __uint_as_float(kw[w] & 0xffff0000u);
                out[w] = A::pack2(k0 * __builtin_amdgcn_exp2f(fmaf(E[8 * kb + 2 * w], unit, cu)),
                                  k1 * __builtin_amdgcn_exp2f(fmaf(E[8 * kb + 2 * w + 1], unit, cu)));
            }
            lds_st<u32x4>(kt_r + kt_buf * F::KT_BYTES + 32 * ct * 64 + kt_p[kb], out);
        }
    };

    // ---- multiplying: U[st][:, 32 ct ..] += K~^T V ----
    f32x16 acc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[dt][j] = 0.f;
    auto multiply = [&](uint32_t v_slot, uint32_t kt_buf) {
        A::Frag vf[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) vf[kb] = rows_frag(sm + F::O_V + v_slot * F::TEN, kb);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
                A::mma(acc[dt], A::load_frag(kt_r + kt_buf * F::KT_BYTES + 32 * dt * 64 + kt_p[kb]), vf[kb]);
    };

    // ---- the walk: interval n prepares step n and multiplies step n - 1 ----
    issue(0, 0, 0);
    if (nsteps > 1) issue(1, 1, 1);
    uint32_t kg_n = 0, v_n = 0;          // slots of step n
    uint32_t kg_i = 2, v_i = 2;          // slots of step n + LEAD
    for (int n = 0; n <= nsteps; ++n) {
        // step n has landed (the loads of step n + 1 may still be in flight); K~ of step n - 1 is complete; the slots
        // and the K~ buffer that this interval overwrites have been read by everyone
        if (n + 1 < nsteps) wait_loads_and_barrier<4>();
        else wait_loads_and_barrier<0>();
        if (n + F::LEAD < nsteps) issue(kg_i, v_i, n + F::LEAD);
        if (n < nsteps) prepare(kg_n, static_cast<uint32_t>(n) & 1u);
        if (n >= 1) multiply(v_n == 0 ? F::V_SLOTS - 1 : v_n - 1, static_cast<uint32_t>(n - 1) & 1u);
        kg_n = kg_n + 1 == F::KG_SLOTS ? 0 : kg_n + 1;
        v_n = v_n + 1 == F::V_SLOTS ? 0 : v_n + 1;
        kg_i = kg_i + 1 == F::KG_SLOTS ? 0 : kg_i + 1;
        v_i = v_i + 1 == F::V_SLOTS ? 0 : v_i + 1;
    }

    // ---- its contribution -> the slot of the next segment; its log2 decay -> its own decay slot ----
    {
        float *dst = a.ws_state + ((slot + slot_step) * 2 + st) * D * D + (4 * g) * D + 32 * ct + ln;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int j = 0; j < 16; ++j) dst[(32 * dt + 8 * (j >> 2) + (j & 3)) * D] = acc[dt][j];
        if (g == 0) a.ws_decay[slot * 2 * D + st * D + 32 * ct + ln] = carry * unit;
    }
}

// What the lists are made from.
struct SegmentListArgs {
    const int32_t *cu, *seq;
    int B, H;
    int64_t segment;             // tokens, where every sequence is cut
    int piece;                   // tokens, where only the long ones are
    int32_t *seg_first, *seg_count, *cut_seq;
    int4 *list_full, *list_pre;
    int cap_full, cap_pre, cap_cut, cap_slot;   // entries; state slots (times H)
    int run_min, run_max;        // only the long sequences are cut: pieces per segment to choose from
    float all_cost;              // us: every sequence cut, where that can be chosen too (0: it cannot)
    int chip;                    // workgroups at a time
    float step, step_full, pre, wg, slot, fixed;   // us: see PrefillCosts
    float margin;                // a cut has to be estimated at less than this part of none
};

// Work lists for packed sequences (one workgroup).  Every sequence in segments of the same length, from its start: list_full =
// every (sequence, segment), list_pre = those with a successor.  Thread t takes a contiguous run of sequences.
__device__ __forceinline__ void list_segments(const SegmentListArgs &a)
{
    __shared__ int4 s_sum[256];
    const int t = threadIdx.x;
    const int per = (a.B + 255) / 256;
    const int b0 = t * per, b1 = (b0 + per < a.B) ? b0 + per : a.B;
    auto length_of = [&](int b) -> int64_t {
        const int sq = a.seq ? a.seq[b] : b;
        return static_cast<int64_t>(a.cu[sq + 1]) - a.cu[sq];
    };
    auto segments_of = [&](int64_t Tb) -> int { return Tb > 0 ? static_cast<int>((Tb + a.segment - 1) / a.segment) : 0; };
    int mine = 0, mine_pre = 0, mine_cut = 0;   // segments, those with a successor, and sequences that have such in this thread's run
    for (int b = b0; b < b1; ++b) {
        const int n = segments_of(length_of(b));
        mine += n;
        mine_pre += n > 1 ? n - 1 : 0;
        mine_cut += n > 1;
    }
    // exclusive sums over the threads (those past the last sequence have nothing)
    s_sum[t] = make_int4(mine, mine_pre, mine_cut, 0);
    __syncthreads();
    int at = 0, at_pre = 0, at_cut = 0;
    const int busy = (a.B + per - 1) / per;
    for (int u = 0; u < (t < busy ? t : busy); ++u) {
        const int4 n = s_sum[u];
        at += n.x;
        at_pre += n.y;
        at_cut += n.z;
    }
    int at_slot = at_pre + at_cut;   // (a sequence in n segments has n slots, a whole one none)
    for (int b = b0; b < b1; ++b) {
        const int64_t Tb = length_of(b);
        const int n = segments_of(Tb);
        a.seg_first[b] = at_slot;
        if (n > 1 && at_cut < a.cap_cut) a.cut_seq[at_cut] = b;
        at_cut += n > 1;
        // the capacities hold whenever the offsets add up to the total the caller gave; offsets that do not
        // must not write past the lists (the segments that do not fit are dropped)
        for (int p = 0; p < n; ++p) {
            const int64_t t0 = p * a.segment, t1 = t0 + a.segment < Tb ? t0 + a.segment : Tb;
            const int4 e = make_int4(b, static_cast<int>(t0), static_cast<int>(t1), n > 1 ? at_slot + p : -1);
            if (at + p < a.cap_full) a.list_full[at + p] = e;
            if (p + 1 < n) {
                if (at_pre < a.cap_pre) a.list_pre[at_pre] = e;
                ++at_pre;
            }
        }
        at += n;
        at_slot += n > 1 ? n : 0;
    }
    if (t == 255) {
        a.seg_first[a.B] = at_slot;
        a.seg_count[0] = at < a.cap_full ? at : a.cap_full;
        a.seg_count[1] = at_pre < a.cap_pre ? at_pre : a.cap_pre;
        a.seg_count[2] = at_cut < a.cap_cut ? at_cut : a.cap_cut;
    }
}

__global__ __launch_bounds__(256) void segment_list_kernel(SegmentListArgs a) { list_segments(a); }

// The lists where only the sequences are cut whose chain of steps would outlast all the work spread over the chip (at most 128
// sequences and 256 segments).  A segment is R pieces, counted from the END of the sequence: what precedes the last full segment - the part that
// the pre-pass has to walk, in pieces so that many workgroups do - is as short as it can be.  Pieces begin at multiples of a step; the first one
// may be shorter.  The lengths are known here and not on the host, so R is chosen here, by the same estimates, with R = 0 (nothing is cut)
// among the choices, and every sequence cut where the host's plan has the room for it; the longest segments come first.
__global__ __launch_bounds__(256) void long_segment_list_kernel(SegmentListArgs a)
{
    constexpr int kMost = 256;
    __shared__ int2 s_len[kMost];   // pieces, steps of 32 tokens
    __shared__ int s_key[kMost], s_n[3][kMost];
    __shared__ float s_cost[kMost];
    __shared__ int4 s_entry[kMost];
    const int t = threadIdx.x, piece = a.piece;
    int Tb = 0;
    if (t < a.B) {
        const int sq = a.seq ? a.seq[t] : t;
        Tb = a.cu[sq + 1] - a.cu[sq];
        if (Tb < 0) Tb = 0;
    }
    s_len[t] = make_int2((Tb + piece - 1) / piece, (Tb + 31) / 32);
    __syncthreads();
    const int choices = a.run_max - a.run_min + 2;
    if (t < choices) {   // thread 0: the cost of nothing cut, thread t: of R = run_min + t - 1
        const int R = t == 0 ? 0 : a.run_min + t - 1;
        int chain = 0, pre = 0, more = 0, steps = 0, sequences = 0;
        for (int b = 0; b < a.B; ++b) {
            const int2 len = s_len[b];
            const bool cut = R > 0 && len.x > R;
            if (cut) {
                more += (len.x - 1) / R;
                pre += len.x - R;
                ++sequences;
            }
            steps += len.y;
            const int longest = cut ? R * (piece / 32) : len.y;
            chain = longest > chain ? longest : chain;
        }
        // The longest chain and all work spread over the chip: the nearer they are, the more the one delays the other (their 4-norm:
        // 20 sequences of up to 8192 tokens, 610 and 474, take 625 us whole)
        const float H = static_cast<float>(a.H) / static_cast<float>(a.chip);
        const float spread = ((a.B + more) * a.wg + steps * a.step_full) * H, alone = a.wg + chain * a.step;
        const float walks = pre * H, s2 = spread * spread, a2 = alone * alone;
        float cost = __builtin_sqrtf(__builtin_sqrtf(s2 * s2 + a2 * a2));
        if (pre > 0) cost += a.fixed + (walks > 1.f ? walks : 1.f) * (piece / 32) * a.pre + a.slot * pre * a.H;
        if (more > (a.cap_full < kMost ? a.cap_full : kMost) - a.B || pre > a.cap_pre || pre + sequences > a.cap_slot) cost = 3.0e38f;   // more than there is room for
        s_cost[t] = cost;
    }
    __syncthreads();
    int R = 0;
    float least = a.margin * s_cost[0];
    for (int u = 1; u < choices; ++u)
        if (s_cost[u] < least) {
            least = s_cost[u];
            R = a.run_min + u - 1;
        }
    if (a.all_cost > 0.f && !((R > 0 ? least : s_cost[0]) < a.all_cost)) {   // (the same for all threads)
        list_segments(a);
        return;
    }
    const int n = (Tb + piece - 1) / piece, ahead = (n * piece - Tb) / 32 * 32;   // pieces, and what the first one is short of
    const bool cut = R > 0 && n > R;
    const int nseg = cut ? (n + R - 1) / R : (Tb > 0 ? 1 : 0), npre = cut ? n - R : 0, nslot = cut ? npre + 1 : 0;
    s_n[0][t] = nseg;
    s_n[1][t] = npre;
    s_n[2][t] = nslot;
    s_key[t] = -1;
    __syncthreads();
    int at = 0, at_pre = 0, at_slot = 0;
    for (int u = 0; u < (t < a.B ? t : a.B); ++u) {
        at += s_n[0][u];
        at_pre += s_n[1][u];
        at_slot += s_n[2][u];
    }
    const int at_cut = at_slot - at_pre;   // (one slot more than pieces each)
    if (cut && at_cut < a.cap_cut) a.cut_seq[at_cut] = t;
    auto begin = [&](int i) { return i > 0 ? i * piece - ahead : 0; };   // of piece i
    if (t <= a.B) a.seg_first[t] = at_slot;                             // (t == B: all slots)
    for (int i = 0; i < npre; ++i) a.list_pre[at_pre + i] = make_int4(t, begin(i), begin(i + 1), at_slot + i);
    for (int k = 0; k < nseg; ++k) {
        const int f = k > 0 ? n - R * (nseg - k) : 0, t0 = begin(f), t1 = k + 1 < nseg ? begin(n - R * (nseg - k - 1)) : Tb;
        s_entry[at + k] = make_int4(t, t0, t1, cut ? at_slot + f : -1);
        s_key[at + k] = (t1 - t0 < (1 << 22) ? t1 - t0 : (1 << 22)) * kMost + (kMost - 1 - at - k);
    }
    if (t == kMost - 1) {
        a.seg_count[0] = at + nseg;
        a.seg_count[1] = at_pre + npre;
        a.seg_count[2] = at_cut;
    }
    __syncthreads();
    if (s_key[t] >= 0) {
        int rank = 0;
        for (int u = 0; u < kMost && u < a.cap_full; ++u) rank += s_key[u] > s_key[t] ? 1 : 0;
        a.list_full[rank] = s_entry[t];
    }
}

// Elementwise scan over the segments of every (sequence, head) that has more than one: s_0 = caller's state goes to
// the slot of segment 0; s_{p+1} = 2^{decay_p} s_p + U_p goes to the slot of segment p+1, where the segment_state
// kernel had left U_p.  The chunk loop then takes every initial state of such a sequence from the slots.
template <int D, int kAhead = 4>
__global__ __launch_bounds__(256) void segment_scan_kernel(const float *__restrict__ S1, const float *__restrict__ S2,
                                                           float *__restrict__ ws_state,
                                                           const float *__restrict__ ws_decay, int BH, int P,
                                                           const int32_t *__restrict__ slot,
                                                           const int32_t *__restrict__ seg_first, const int32_t *__restrict__ seg_count,
                                                           const int32_t *__restrict__ cut_seq, int H, int zero_init, int beta)
{
    // one thread per 4 adjacent columns of one (bh, state, row); a workgroup has part of one (bh, state) only
    constexpr int kParts = D * (D / 4) / 256;
    const int bi = static_cast<int>(blockIdx.x / kParts);   // bh*2 + i
    const int in_state = static_cast<int>(blockIdx.x % kParts) * 256 + static_cast<int>(threadIdx.x);
    const int c4 = in_state % (D / 4), row = in_state / (D / 4);
    const int i = bi & 1, bh = bi >> 1;
    if (beta && i) return;   // beta mode: one state; the second slot of decays holds the log2 decays of its columns
    const int h = bh % H;
    int b = bh / H;
    size_t slot0 = bh, slot_step = BH;
    if (seg_first) {   // work lists: b of the sequences that are cut
        if (b >= seg_count[2]) return;
        b = cut_seq[b];
        P = seg_first[b + 1] - seg_first[b];
        slot0 = static_cast<size_t>(seg_first[b]) * H + h;
        slot_step = H;
    }
    if (P <= 1) return;
    const size_t sbh = static_cast<size_t>(slot ? slot[b] : b) * H + h;
    const float *src = (i ? S2 : S1) + (sbh * D + row) * D + c4 * 4;
    float4 s = zero_init ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<const float4 *>(src);
    const size_t in_slot = (static_cast<size_t>(i) * D + row) * D + c4 * 4;   // this thread's place inside a slot
    auto decay_of = [&](int p) { return ws_decay + (slot0 + p * slot_step) * 2 * D; };
    auto state_of = [&](int p) { return reinterpret_cast<float4 *>(ws_state + (slot0 + p * slot_step) * 2 * D * D + in_slot); };
    // Latency where there are few heads: a segment's loads wait for nothing, but the compiler cannot move them ahead of the store of
    // the one before.  Those of 4 segments go out together: a call of 300 tokens and 4 heads, d = 64, fp32 takes 22.1 us instead of
    // 23.6, 16384 tokens of 32 heads, d = 128, bf16 268 instead of 271.  With 8 at a time no more (22.1), and 115 registers, not 63.
    // 32 heads, d = 128 and six segments are bound by HBM: 25 MB read and written in 9 us.
    for (int p = 0; p + 1 < P; p += kAhead) {
        float dr[kAhead];
        float4 dc[kAhead], x[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            if (p + j + 1 >= P) break;
            dr[j] = decay_of(p + j)[i * D + row];
            if (beta) dc[j] = *reinterpret_cast<const float4 *>(decay_of(p + j) + D + c4 * 4);
            x[j] = *state_of(p + j + 1);
        }
        if (p == 0 && !zero_init) *state_of(0) = s;   // zero states: segment 0 starts from registers set to zero
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            if (p + j + 1 >= P) break;
            float4 dec = make_float4(dr[j], dr[j], dr[j], dr[j]);
            if (beta) {
                dec.x += dc[j].x; dec.y += dc[j].y; dec.z += dc[j].z; dec.w += dc[j].w;
            }
            dec.x = __builtin_amdgcn_exp2f(dec.x); dec.y = __builtin_amdgcn_exp2f(dec.y);
            dec.z = __builtin_amdgcn_exp2f(dec.z); dec.w = __builtin_amdgcn_exp2f(dec.w);
            s.x = fmaf(dec.x, s.x, x[j].x);
            s.y = fmaf(dec.y, s.y, x[j].y);
            s.z = fmaf(dec.z, s.z, x[j].z);
            s.w = fmaf(dec.w, s.w, x[j].w);
            if (!(zero_init && p + j == 0)) *state_of(p + j + 1) = s;   // from zero states the first slot already holds its result
        }
    }
}


// Workgroups of the chunk loop that the chip holds at one time: two per compute unit at d = 64 with 16-bit io, else one (LDS).
int chip_slots(const dsla_desc &d) { return d.d_k == 64 && d.io_dtype == DSLA_BF16 ? 512 : 256; }

// Estimates (us): a step of 32 tokens where the chain of one workgroup counts / where every compute unit is busy, a step of
// the pre-pass, what a workgroup costs besides its steps, a state slot written, scanned and read again, the lists of a packed
// batch and the scan besides its slots.
struct PrefillCosts {
    double step, step_full, pre, wg, slot, lists;
    double step_alone;   // a step where no compute unit has two workgroups
};
PrefillCosts prefill_costs(const dsla_desc &d)
{
    const bool f32 = d.io_dtype == DSLA_F32, small = d.d_k == 64, preact = d.gate_mode == DSLA_GATE_PREACT;
    PrefillCosts c;
    c.step = f32 ? (small ? 4.5 : 11.1) : (small ? (preact ? 1.8 : 1.4) : (preact ? 2.35 : 2.0));
    c.step_alone = f32 && small ? 3.6 : c.step;   // (launch_f32)
    c.step_full = f32 ? c.step : (small ? 2.5 : (preact ? 3.4 : 2.9));
    c.pre = f32 ? (small ? 2.2 : 5.1) : (small ? 1.2 : (preact ? 2.1 : 1.5));
    c.wg = f32 ? (small ? 3.0 : 5.0) : (small ? 5.0 : 8.0);
    c.slot = f32 ? (small ? 0.028 : 0.06) : (small ? 0.04 : 0.05);
    c.lists = f32 ? (small ? 5.0 : 4.0) : (small ? 9.0 : 6.0);
    return c;
}
// All work spread over the chip takes this part of what step_full says (which stays, for the rules that were measured with it).
constexpr double kSpread = 0.92;

// F32Kern with or without roles.  With them (d = 64) a compute unit holds one workgroup, so they are taken where every workgroup has
// a unit to itself.  Without / with, us, 600 tokens in one segment: 256 heads 109 / 91; past one
// to a unit 288 heads 157 / 164, 512 heads 165 / 173, 2048 heads of 512 tokens 535 / 573.
// (The caller takes the launch's error: hipGetLastError() answers only once.)
template <int D, class TG, bool kFull>
void launch_f32(unsigned grid, const PrefillArgs &a, ProfileScope &ps, hipStream_t stream)
{
    if constexpr (D == 64) {
        if (grid <= 256) {
            DSLA_LAUNCH(ps, (prefill_f32_kernel<D, TG, kFull, true>), dim3(grid), dim3(F32Kern<D, TG, kFull, true>::NT), 0, stream, a);
            return;
        }
    }
    DSLA_LAUNCH(ps, (prefill_f32_kernel<D, TG, kFull, false>), dim3(grid), dim3(F32Kern<D, TG, kFull, false>::NT), 0, stream, a);
}

template <int D, class TIO, class TG, bool kExt, bool kBeta = false>
hipError_t launch_x(const dsla_desc &d, const PrefillPlan &plan, PrefillArgs &a, hipStream_t stream)
{
    const int BH = d.B * d.H;
    // The pre-pass and the scan see every segment but the last as R pieces (R = plan.pre_split; 1 with work lists):
    // to them the sequence has R (P - 1) + 1 segments of segment_tokens / R tokens, the last one longer, which neither
    // of them touches.  The chunk loop then finds the state entering its segment p in slot R p.
    const int R = plan.segments > 1 ? plan.pre_split : 1;
    PrefillArgs af = a;
    af.P = R * (plan.segments - 1) + 1;
    af.seg_tokens = a.seg_tokens / R;
    a.slot_mul = R;
    // workgroups of the two big kernels: one per (segment, sequence, head); with work lists one per (list entry, head)
    const unsigned grid_pre = a.list_full ? static_cast<unsigned>(plan.max_pre_items * d.H)
                                          : static_cast<unsigned>(BH * (af.P - 1));
    const unsigned grid_full = a.list_full ? static_cast<unsigned>(plan.max_items * d.H)
                                           : static_cast<unsigned>(BH * plan.segments);
    hipError_t err = hipSuccess;
    if (plan.segments > 1) {
        if (a.list_full) {
            ProfileScope ps(DSLA_KERNEL_PREFILL_SEGMENT_LIST, stream);
            const PrefillCosts c = prefill_costs(d);
            SegmentListArgs l;
            l.cu = a.cu;
            l.seq = a.seq;
            l.B = d.B;
            l.H = d.H;
            l.segment = a.seg_tokens;
            l.piece = plan.long_piece;
            l.all_cost = plan.all_cost;
            l.seg_first = const_cast<int32_t *>(a.seg_first);
            l.seg_count = const_cast<int32_t *>(a.seg_count);
            l.cut_seq = const_cast<int32_t *>(a.cut_seq);
            l.cap_cut = static_cast<int>(plan.max_cut);
            l.list_full = const_cast<int4 *>(a.list_full);
            l.list_pre = const_cast<int4 *>(a.list_pre);
            l.cap_full = static_cast<int>(plan.max_items);
            l.cap_pre = static_cast<int>(plan.max_pre_items);
            l.cap_slot = static_cast<int>(plan.all_cost > 0.f ? plan.max_items : plan.max_pre_items);
            l.run_min = plan.run_min;
            l.run_max = plan.run_max;
            l.chip = chip_slots(d);
            l.step = static_cast<float>(c.step);
            l.step_full = static_cast<float>(kSpread * c.step_full);
            l.pre = static_cast<float>(c.pre);
            l.wg = static_cast<float>(c.wg);
            l.slot = static_cast<float>(c.slot);
            l.fixed = static_cast<float>(2 * c.wg + c.lists);
            l.margin = d.d_k == 64 ? 0.92f : 0.98f;   // (two workgroups to a compute unit are harder to estimate)
            if (plan.run_max > 0) DSLA_LAUNCH(ps, long_segment_list_kernel, dim3(1), dim3(256), 0, stream, l);
            else DSLA_LAUNCH(ps, segment_list_kernel, dim3(1), dim3(256), 0, stream, l);
            err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        if (grid_pre > 0) {
            ProfileScope ps(DSLA_KERNEL_PREFILL_SEGMENT_STATE, stream);
            // the pre-pass of its own design where it is built; its per-lane offsets inside a step are 32-bit
            constexpr bool kFast = D == SegFast::D && std::is_same<TIO, bf16_t>::value && std::is_same<TG, bf16_t>::value && !kBeta;
            if constexpr (std::is_same<TIO, float>::value && !kBeta)
                launch_f32<D, TG, false>(grid_pre, af, ps, stream);
            else if (kFast && static_cast<int64_t>(d.H) * D * 2 * SegFast::S < (int64_t{1} << 31))
                DSLA_LAUNCH(ps, segment_state_fast_kernel, dim3(grid_pre), dim3(SegFast::NT), 0, stream, af);
            else
                DSLA_LAUNCH(ps, (prefill_kernel<D, TIO, TG, false, kExt, kBeta>), dim3(grid_pre), dim3(4 * D), 0, stream, af);
            err = hipGetLastError();
        }
        if (err != hipSuccess) return err;
        {
            ProfileScope ps(DSLA_KERNEL_PREFILL_SEGMENT_SCAN, stream);
            const int n_scan = a.list_full ? static_cast<int>(plan.max_cut) * d.H : BH;   // (sequence, head)
            DSLA_LAUNCH(ps, (segment_scan_kernel<D>), dim3(static_cast<unsigned>(n_scan) * 2 * (D * (D / 4) / 256)), dim3(256), 0,
                               stream, a.S1, a.S2, a.ws_state, a.ws_decay, n_scan, af.P, a.slot, a.seg_first, a.seg_count, a.cut_seq, a.H,
                               a.zero_init, kBeta ? 1 : 0);
            err = hipGetLastError();
        }
        if (err != hipSuccess) return err;
    }
    {
        ProfileScope ps(DSLA_KERNEL_PREFILL_CHUNK_LOOP, stream);
        if constexpr (std::is_same<TIO, float>::value && !kBeta)
            launch_f32<D, TG, true>(grid_full, a, ps, stream);
        else
            DSLA_LAUNCH(ps, (prefill_kernel<D, TIO, TG, true, kExt, kBeta>), dim3(grid_full), dim3(4 * D), 0, stream, a);
    }
    err = hipGetLastError();
    return err;
}

// Ordinary launches keep the lean kernels; explicit blend coefficients, grouped key/value heads and accumulation
// into o select the extended ones.
template <int D, class TIO, class TG>
hipError_t launch_t(const dsla_desc &d, const PrefillPlan &plan, PrefillArgs &a, hipStream_t stream)
{
    if (a.beta) return launch_x<D, TIO, TG, true, true>(d, plan, a, stream);
    if constexpr (std::is_same<TIO, float>::value) return launch_x<D, TIO, TG, true>(d, plan, a, stream);   // (F32Kern is one for all of them)
    else if (a.explicit_w || a.accumulate || a.Hkv != a.H) return launch_x<D, TIO, TG, true>(d, plan, a, stream);
    else return launch_x<D, TIO, TG, false>(d, plan, a, stream);
}

template <int D, class TIO>
hipError_t launch_g(const dsla_desc &d, const PrefillPlan &plan, PrefillArgs &a, hipStream_t stream)
{
    if (d.gate_dtype == DSLA_BF16) return launch_t<D, TIO, bf16_t>(d, plan, a, stream);
    return launch_t<D, TIO, float>(d, plan, a, stream);
}

// The chunk length only sets the granularity of the segment split; the kernels step through 32 tokens at a time.
bool combo_built(int D, int C, int io)
{
    return (io == DSLA_BF16 || io == DSLA_F32) && (D == 64 || D == 128) && (C == 32 || C == 64 || C == 128);
}

}  // namespace

namespace {
// Fills the plan from the chunk length, the number of segments P the longest sequence is cut into, and its length.
void finish_plan(const dsla_desc &d, int C, int64_t P, int64_t nchunks, bool may_split, PrefillPlan *plan)
{
    const int D = d.d_k;
    const int64_t BH = static_cast<int64_t>(d.B) * d.H;
    if (P < 1) P = 1;
    if (P > nchunks) P = nchunks;
    const int64_t cps = (nchunks + P - 1) / P;
    P = (nchunks + cps - 1) / cps;
    plan->chunk = C;
    plan->segments = static_cast<int>(P);
    plan->segment_tokens = cps * C;
    plan->state_elems = static_cast<size_t>(BH) * D * D;
    plan->max_items = plan->max_pre_items = 0;
    plan->longest_first = false;
    plan->run_min = plan->run_max = plan->long_piece = 0;
    plan->all_cost = 0.f;
    plan->max_cut = 0;
    plan->ws_lists_bytes = 0;
    // The pre-pass has one workgroup per (segment but the last, sequence, head).  With two segments that is at most
    // half of the compute units (65 .. 128 heads in all; short sequences): it then works on the two halves of the first
    // segment and the scan combines them: measured at B H = 128, T = 16384 the pre-pass streams at 3.7 TB/s from 128
    // workgroups and at 5.7 TB/s from 256.  With more segments the longer scan costs what the shorter pieces gain
    // (B H = 32, T = 1024, four segments: pre-pass - 2 us, scan + 5 us).  A caller who names the number of segments
    // gets exactly those.
    plan->pre_split = (may_split && P == 2 && cps % 2 == 0 && cps * C >= 256 && BH * 2 <= ((D == 64) ? 512 : 256)) ? 2 : 1;
    if (P > 1) {
        const int64_t pieces = plan->pre_split * (P - 1) + 1;
        plan->ws_state_bytes = static_cast<size_t>(pieces) * plan->state_elems * 2 * sizeof(float);
        plan->ws_decay_bytes = ((static_cast<size_t>(pieces - 1) * BH * 2 * D * sizeof(float)) + 255) / 256 * 256;
    } else {
        plan->ws_state_bytes = 0;
        plan->ws_decay_bytes = 0;
    }
    plan->ws_total_bytes = plan->ws_ask_bytes = plan->ws_need_bytes = plan->ws_state_bytes + plan->ws_decay_bytes;
}
int plan_chunk(const dsla_desc &d)
{
    if (d.d_k != d.d_v) return 0;
    int C = d.chunk;
    if (C == 0) C = combo_built(d.d_k, 64, d.io_dtype) ? 64 : 32;
    return combo_built(d.d_k, C, d.io_dtype) ? C : 0;
}
}  // namespace

namespace {
// The figures by which a packed call without its buffer is refused or runs whole.  They are part of what callers rely on: they stay
// when kernels get faster and the estimates follow.
PrefillCosts refusal_costs(const dsla_desc &d)
{
    const bool f32 = d.io_dtype == DSLA_F32, small = d.d_k == 64, preact = d.gate_mode == DSLA_GATE_PREACT;
    PrefillCosts c;
    c.step = f32 ? (small ? 7.0 : 16.0) : (small ? (preact ? 1.8 : 1.4) : (preact ? 2.35 : 2.0));
    c.step_alone = c.step;
    c.step_full = f32 ? c.step : (small ? 2.5 : (preact ? 3.4 : 2.9));
    c.pre = f32 ? c.step / 3 : (small ? 1.2 : (preact ? 2.1 : 1.5));
    c.wg = f32 ? (small ? 7.0 : 16.0) : (small ? 5.0 : 8.0);
    c.slot = f32 ? (small ? 0.025 : 0.06) : (small ? 0.04 : 0.05);
    c.lists = f32 ? (small ? 5.0 : 4.0) : (small ? 9.0 : 6.0);
    return c;
}
}  // namespace

namespace {
// Estimate (us) of a dense fp32 call by its plan.  Estimated / measured: 256 tokens in four segments, d = 64, 4 and 32 heads 21.1 / 22.6 and
// 24.3 / 24.8, d = 128, 8 and 32 heads 48 / 47 and 54 / 53; 512 tokens in two 47 / 47 and 123 / 124; whole, d = 64, 64 and 128 tokens 10.2 / 11.2 and 17.4 / 18.4, d = 128, 64 tokens 27.2 / 27.3.
double plan_cost(const dsla_desc &d, const PrefillPlan &plan, int64_t T)
{
    const PrefillCosts c = prefill_costs(d);
    const double groups = static_cast<double>(d.B) * d.H * plan.segments, rounds = groups > 256 ? groups / 256 : 1.0;
    const double steps = static_cast<double>(((T < plan.segment_tokens ? T : plan.segment_tokens) + 31) / 32);
    if (plan.segments == 1) return c.wg + rounds * steps * (groups > 256 ? c.step / 1.3 : c.step_alone);
    return c.wg + (d.d_k == 64 ? 6.1 : 9.1) + rounds * steps * (c.pre / plan.pre_split + c.step_alone) + c.slot * groups;
}
}  // namespace

bool prefill_plan(const dsla_desc &d, int64_t T, PrefillPlan *plan, size_t available)
{
    const int C = plan_chunk(d);
    if (!C) return false;
    const int64_t nchunks = (T + C - 1) / C;
    const int64_t BH = static_cast<int64_t>(d.B) * d.H;
    int64_t P, P_coarse = 0;
    if (d.segments > 0) {
        P = d.segments;
    } else {
        // Enough workgroups to cover the chip, but at least 4 chunks per segment ...
        const int64_t target = (d.d_k == 64) ? 512 : 256;
        P = target / BH;
        if (P > nchunks / 4) P = nchunks / 4;
        P_coarse = P < 1 ? 1 : P;
        // ... or fewer where that leaves the chip idle (plans of one or two segments stay as they are in 16 bits: there
        // the pre-pass and the scan cost what the shorter segments gain).  A step of 32 tokens takes 2 us in 16-bit
        // arithmetic however few workgroups run, in fp32 3.6 us (d = 64) and 11 us (d = 128), a segment's share of the
        // pre-pass half of that, pre-pass and scan about 6 to 9 us more.  Measured in us at 1000 tokens with 4, 3, 2 chunks per
        // segment: bf16, 32 heads, d = 128 47, 43, 47; 8 heads 43, 38, 36; 4 heads, d = 64 35, 30, 27; fp32, 32 heads, d = 128
        // 165, 132, 108; fp32, 4 heads, d = 64, 256 tokens whole and with 2, 1 chunks: 39, 36, 24.
        const bool f32 = d.io_dtype == DSLA_F32;
        // 256 heads of 1000, 2000, 8000 tokens, d = 64, whole / in two: 54 / 71, 104 / 156, 382 / 602; 160 heads whole / in three: 52 / 62, 127 / 135, 365 / 394
        if (!f32 && d.d_k == 64 && BH > 128) P = P_coarse = 1;
        // 16 bits, 257 to 704 tokens: neither of the rules above fits (the first makes one or two segments, at two of which half of the
        // chip idles through a pre-pass of its own length).  Whole, or one to three chunks per segment, by estimates (us) fitted
        // to 64 .. 704 tokens; a finer cut has to be 7 % ahead.  Two segments / this: d = 128, 4 heads of 520 and 700 tokens 42.5 / 25.6,
        // 42.4 / 28.7; 32 heads 45.5 / 36.1 and 46.0 / 38.5; 96 heads, now whole, 54.6 / 41.0 and 60.1 / 50.4; d = 64, 32 heads
        // 37.3 / 26.8 and 36.6 / 28.0; whole / this: d = 128, 4 heads of 400 tokens 30.7 / 24.0.  (A caller's chunk of 128 keeps its
        // granularity.)  One chunk per segment only with few workgroups: d = 128, 16 heads of 378 tokens 31.0, whole 29.0.
        // More than 85 heads fill a third of the chip and more by themselves: a cut saves the less per step the more heads there
        // are, and costs 13 to 20 us whatever their number.  In two / whole (d = 128): 96 heads of 710, 1100, 1500 tokens 61.5 / 52.5,
        // 86 / 75, 92 / 95; 128 heads of 710, 1500, 3000 71.5 / 53.8, 119 / 99, 194 / 184; d = 64, in four or five / whole: 96 heads of
        // 710, 1300 41.4 / 37.1, 59 / 62; 128 heads of 710, 1500, 2200 45.2 / 37.6, 77 / 71, 100 / 101.
        // Per step a whole prompt loses 0.48 (d = 128: 0.43) us at 96 heads and less by 0.29 (0.33) for 32 more, but not less than a
        // floor: past 110 heads their number hardly counts.  At d = 128, where the cut is in two, it costs least where the pre-pass works on
        // the halves of the first segment (an even number of chunks), and less from zero states.  Cut / whole: d = 128, 128 heads of 3267 tokens 193 / 233, of 1959
        // (halves) 127 / 138, of 2572 (none) 1.00, 120 of 2709 as pre-activations (halves) 170 / 205, 104 of 1491 (halves) 87 / 97, of 1589
        // (none) as pre-activations 0.91; d = 64, 128 heads of 1651 69 / 77, 112 of 1232 1.07.
        const double heads = static_cast<double>(BH - 96) / 32, steps_d = static_cast<double>(T) / 32;
        const bool gates32 = d.gate_dtype != DSLA_BF16, preacts = d.gate_mode == DSLA_GATE_PREACT;
        const int64_t half = (nchunks + 1) / 2;   // chunks per segment of a cut in two
        const double loss = d.d_k == 64 ? std::max(0.48 - 0.29 * heads, preacts ? 0.33 : (gates32 ? 0.24 : 0.36))
                                        : std::max(0.43 - 0.33 * heads, gates32 ? 0.28 : (preacts ? 0.30 : 0.25));
        double costs;   // (us; 32-bit gates go through the general pre-pass)
        if (d.d_k == 64) costs = preacts ? (gates32 ? 12.3 : 11.2) : (gates32 ? 15.5 : 13.2);
        else if (half % 2 != 0) costs = gates32 ? (d.zero_init ? 24.0 : 28.0) : 20.0;
        else if (gates32) costs = preacts ? (d.zero_init ? 15.5 : 20.0) : (d.zero_init ? 16.5 : 25.0);
        else costs = d.zero_init ? 12.0 : 13.2;
        if (!f32 && C <= 64 && T > 704 && BH > 85 && BH <= 128 && steps_d * loss < costs) {
            P = 1;
        } else if (!f32 && C <= 64 && T > 256 && T <= 704) {
            const bool small = d.d_k == 64, preact = d.gate_mode == DSLA_GATE_PREACT;
            const double step = (small ? 1.37 : 1.81) + (preact ? 0.48 : 0.0), pre = (small ? 1.2 : 1.3) + (preact ? 0.3 : 0.0);
            const double fixed = small ? 6.8 : 7.0, slot = small ? 0.026 : 0.057, wg = small ? 5.6 : 7.5;
            double best = wg + static_cast<double>((T + 31) / 32) * step;
            P = 1;
            for (int64_t tokens = 192; tokens >= 64; tokens -= C) {   // (chunks of 32: also the lengths between)
                const int64_t parts = (T + tokens - 1) / tokens, longest = (nchunks + parts - 1) / parts * C;   // as finish_plan evens them out
                if (BH * parts > (tokens > 64 ? 256 : (small ? 160 : 64))) break;
                const double cut = wg + fixed + static_cast<double>(longest / 32) * (step + pre) + slot * static_cast<double>(BH * parts);
                if (cut < 0.93 * best) {
                    best = cut;
                    P = parts;
                }
            }
        } else if (P >= 3 || (f32 && (P < 2 || BH * P > chip_slots(d)))) {
            const int64_t most = chip_slots(d) / BH;
            const int64_t least = f32 ? 1 : (BH * ((nchunks + 1) / 2) <= 128 ? 2 : 3);   // chunks per segment
            auto chunks_of = [&](int64_t segments_at_most) {
                const int64_t cps = segments_at_most > 0 ? (nchunks + segments_at_most - 1) / segments_at_most : nchunks;
                return cps < least ? least : cps;
            };
            int64_t cps = chunks_of(most);
            // Two workgroups on a compute unit take 1.7 times as long as one: either every segment has a unit to itself, or
            // they are as short as two to a unit allow.  d = 64, segments of one / two to a unit: 24 heads of 2500 tokens 41 / 46,
            // 60 of 1000 39 / 42, 8 of 8000 54 / 61; 24 of 4000 59 / 55, 60 of 1500 49 / 47.
            if (chip_slots(d) == 512 && 10 * chunks_of(256 / BH) <= 17 * cps) cps = chunks_of(256 / BH);
            // fp32, short: the cut saves steps of the chain and costs the pre-pass, its launches and the slots (us, whole / in
            // segments of one chunk: 128 tokens, d = 64, 4 heads 18.7 / 21.8, 64 heads 19.4 / 25.0; 160 tokens, 4 heads 22.2 / 22.4, 32
            // heads 22.7 / 24.3; 180 tokens, 4 heads 25.8 / 22.6, 64 heads 26.4 / 27.5; 128 tokens, d = 128, 8 heads 49.4 / 46.0, 32 heads
            // 50.3 / 51.2, 96 heads 53.6 / 60.8; 180 tokens, 32 heads 72.2 / 53.7)
            if (f32 && P < 2) {
                const PrefillCosts c = prefill_costs(d);
                const int64_t steps = (T + 31) / 32, chain = cps * C / 32 < steps ? cps * C / 32 : steps;
                const double launches = d.d_k == 64 ? 6.1 : 9.1;
                if (static_cast<double>(steps - chain) * c.step_alone <= chain * c.pre + launches + c.slot * BH * ((nchunks + cps - 1) / cps))
                    cps = nchunks;
            }
            P = (nchunks + cps - 1) / cps;
            if (most <= 1) P_coarse = 1;
        }
    }
    finish_plan(d, C, P, nchunks, d.segments <= 0, plan);
    if (P_coarse > 0 && P_coarse != P) {
        // The first rule's cut needs other numbers of slots at other lengths.  The size query covers both, and a call takes the
        // first rule's where only that one fits: a buffer sized for a longer sequence may hold fewer slots than
        // this one would fill, and has to serve it all the same.
        PrefillPlan coarse;
        finish_plan(d, C, P_coarse, nchunks, true, &coarse);
        const size_t ask = coarse.ws_total_bytes > plan->ws_total_bytes ? coarse.ws_total_bytes : plan->ws_total_bytes;
        if (plan->ws_total_bytes > available && coarse.ws_total_bytes <= available) *plan = coarse;
        // Whole where the coarse cut needs a buffer: the caller brings that buffer all the same (it is what the size query asks for).
        // In 16 bits a cut where the coarse plan is whole is an offer: a call without a buffer that it can use runs whole.
        if (P == 1 && coarse.ws_total_bytes > available) *plan = coarse;
        if (P == 1) plan->ws_need_bytes = coarse.ws_total_bytes;
        else if (P_coarse == 1 && d.io_dtype == DSLA_BF16) plan->ws_need_bytes = 0;
        plan->ws_ask_bytes = ask;
    }
    return true;
}

namespace {
// Do whole packed sequences go longest first?  Every workgroup pays for its rank (about 2 us and 1 more per 128 sequences),
// so with R rounds of workgroups the call pays R times, and it gains at most a part of the longest chain, which no longer
// starts late; max_T may bound the lengths loosely, and then there is nothing to gain: the rank also has to be small
// against an average workgroup.  Own order / longest first (us, d = 128, 32 heads): 16 sequences of 1 to 600 tokens
// 57 / 46, 32 of 1 to 2500 151 / 134, 48 of 64 to 1000 216 / 207, 64 of those 467 / 476; 8 heads: 128 of 1 to 2500
// 211 / 158.  Not taken: 48 of up to 40 and one of 300 86 / 101 (512: 950 / 1390), 256 of 1 to 600 658 / 752.  Up to 256
// tokens it never paid.
bool order_pays(const dsla_desc &d, int64_t total_T, int64_t max_T)
{
    const double rounds = static_cast<double>(d.B) * d.H / chip_slots(d), rank = 2.0 + d.B / 128.0;
    if (d.B < 2 || d.B > 4 * d.d_k || max_T <= 256 || rounds <= 1.0) return false;   // a thread per sequence
    const PrefillCosts c = prefill_costs(d);
    const double longest = static_cast<double>(max_T) / 32, mean = static_cast<double>(total_T) / 32 / d.B;
    return longest * c.step >= 2.4 * rounds * rank && c.wg + mean * c.step_full >= 2.5 * rank;
}
}  // namespace

namespace {
size_t lists_bytes(const dsla_desc &d, const PrefillPlan &p)
{
    auto up = [](size_t n) { return (n + 255) / 256 * 256; };
    return up((static_cast<size_t>(d.B) + 1) * 4) + up((static_cast<size_t>(d.B) + 4) * 4) + up(p.max_items * 16) + up(p.max_pre_items * 16);
}

constexpr double kOfferLong = 400;   // us: see below

// A batch that stays whole because cutting everything costs more than it saves, but whose longest sequences outlast all its work
// spread over the chip: these alone are cut (long_segment_list_kernel decides where, and whether).  It takes the lists, a pre-pass over the
// beginnings of the long sequences and a scan.  Whole / cut, 32 heads, d = 128: 20 sequences of up to 8192 tokens as pre-activations 635 / 532 us, with
// log-gates 578 / 473.  Not at d = 64, where a compute unit's second workgroup slows the first one's chain, which no estimate here knows: 32 of up to
// 6768 tokens 430 / 350, but 8 of up to 7301 338 / 413.
// max_T may bound the lengths loosely and then nothing is cut: the lists, an empty pre-pass and an empty scan take 10 us (5 to 16, less what the ranks
// of whole sequences would take).  So only where all work spread over the chip, which the call takes at least, is kOfferLong or more: nothing cut / whole,
// 32 heads, d = 128: 22 sequences of up to a quarter of max_T 434 / 430 us, 39 of up to a half 427 / 420, 10 of those 498 / 487; below, 1.03 at 300 us, 1.05 at 200, 1.2 at 50.
// (What that gives up: 23 of up to 5826 tokens 390 us and not 287.)
// Its slots are as many as `bytes` hold (what the size query answers, or less that a caller brings): the device keeps to them.
// Where cutting every sequence pays (all_cost: its estimate), the long ones alone are one more choice, inside the buffer and the launches of
// cutting all.  How many are long is not known here, and few slots for many long ones make long segments, so the device may also choose to
// cut all: chosen here as if two sequences were the longest, 7 of up to 6913 tokens (8 heads) took 348 us and not 289, 9 of up to 7898 351 and 320,
// d = 64, 4 heads, 22 of up to 4078 131 and 105.  All cut / this: 16 of up to 5451 (8 heads) 361 / 277, 28 of up to 1769 with max_T 7076 (none is cut) 281 / 160.
// The list kernel that chooses takes 3 us more where all are cut in the end, so it has to be worth it for sequences of the same length too; at
// d = 64, where two workgroups share a compute unit and chains take longer than estimated, by far.
void cut_long(const dsla_desc &d, int64_t total_T, int64_t max_T, size_t bytes, double all_cost, PrefillPlan *plan)
{
    if (d.io_dtype == DSLA_F32 || d.B < 2 || d.B > 128 || (d.d_k == 64 && !(all_cost > 0))) return;
    const PrefillCosts c = prefill_costs(d);
    const double H = static_cast<double>(d.H) / chip_slots(d);
    const double spread = (static_cast<double>(d.B) * c.wg + static_cast<double>(total_T) / 32 * kSpread * c.step_full) * H;
    auto both = [&](int64_t steps) { return std::sqrt(std::hypot(spread * spread, (c.wg + steps * c.step) * (c.wg + steps * c.step))); };
    if (!(all_cost > 0) && spread < kOfferLong) return;
    PrefillPlan p = *plan;
    const int64_t piece = max_T >= 4096 ? 512 : 256;   // (a multiple of every chunk)
    p.run_min = static_cast<int>(0.8 * (spread - c.wg) / c.step * 32 / static_cast<double>(piece));
    if (p.run_min < 2) p.run_min = 2;
    const int64_t most = (max_T + piece - 1) / piece - 1;   // pieces per segment that still cut the longest
    if (most < p.run_min) return;
    p.run_max = static_cast<int>(most < p.run_min + 200 ? most : p.run_min + 200);
    // the device's estimate as if two sequences were the longest: has to be below that of the whole batch
    double least = 1e30;
    for (int64_t R = p.run_min; R <= p.run_max; ++R) {
        const double pieces = 2.0 * static_cast<double>(most + 1 - R), walks = pieces * H;
        const double cost = both(R * piece / 32) + 2 * c.wg + c.lists + (walks > 1 ? walks : 1) * (piece / 32) * c.pre + c.slot * pieces * d.H;
        if (cost < least) least = cost;
    }
    if (least > (all_cost > 0 ? 0.78 * all_cost : 0.95 * both((max_T + 31) / 32))) return;
    p.long_piece = static_cast<int>(piece);
    if (all_cost > 0) {
        if (both((total_T / d.B + 31) / 32) > (d.d_k == 64 ? 0.65 : 0.92) * all_cost) return;
        p.all_cost = static_cast<float>(all_cost);
        *plan = p;
        return;
    }
    p.segments = 2;
    p.segment_tokens = piece;
    p.pre_split = 1;
    // n sequences of more than run_min pieces hold at most so many pieces past their last segments; all make `cuts` further segments at most
    const int64_t run = p.run_min * piece, cuts = total_T / run;
    int64_t slots = 0;   // a sequence has one more slot than pieces past its last segment
    for (int64_t n = 1; n <= cuts; ++n) {
        const int64_t tokens = (n * max_T < total_T ? n * max_T : total_T) - n * run;
        if (tokens > 0 && tokens / piece + 2 * n > slots) slots = tokens / piece + 2 * n;
    }
    p.max_items = d.B + cuts;
    p.max_cut = cuts < d.B ? cuts : d.B;
    const size_t slot_bytes = static_cast<size_t>(d.H) * 2 * d.d_k * (d.d_k + 1) * sizeof(float);
    p.max_pre_items = slots;
    const size_t fixed = lists_bytes(d, p) + 256;
    if (p.max_items > 256 || bytes < fixed + 2 * slot_bytes) return;
    const int64_t fit = static_cast<int64_t>((bytes - fixed) / slot_bytes);
    if (fit < slots) slots = fit;
    p.max_pre_items = slots;
    p.ws_state_bytes = static_cast<size_t>(slots) * d.H * 2 * d.d_k * d.d_k * sizeof(float);
    p.ws_decay_bytes = (static_cast<size_t>(slots) * d.H * 2 * d.d_k * sizeof(float) + 255) / 256 * 256;
    p.ws_lists_bytes = lists_bytes(d, p);
    p.ws_total_bytes = p.ws_state_bytes + p.ws_decay_bytes + p.ws_lists_bytes;
    p.longest_first = false;
    *plan = p;
}
}  // namespace

// Where every sequence is cut, packed sequences of different lengths share one segment length; a sequence of length T_b has
// ceil(T_b / segment_tokens) segments (only the long ones cut: cut_long).  The segment length is chosen so that all sequences together make
// about one workgroup per compute unit, the same rule as above on the total instead of a common length (measured on
// mixed batches: twice as many segments gain on some mixes and lose on others, within 10 %).  Whether they are cut is a
// matter of estimates (us): whole sequences take as long as the longest one or as all of them spread over the chip; cut
// ones pay the lists, the pre-pass and the scan for shorter chains.  Measured whole / cut: 40 sequences of up to 651
// tokens (32 heads, d = 128) 127 / 180; 20 of up to 8192 659 / 742; 11 of up to 956 (d = 64) 63 / 78; 8 sequences, one of
// 1900 tokens and 7 short ones 129 / 84; 22 of up to 4015 tokens with 8 heads 257 / 94.
// The kernels find their work in lists built on the device (the lengths are not known here); list and workspace
// sizes are worst cases: sum_b ceil(T_b / L) <= total_T / L + B segments, of which at most total_T / L have a
// successor.
bool prefill_plan_varlen(const dsla_desc &d, int64_t total_T, int64_t max_T, PrefillPlan *plan, size_t available)
{
    const int C = plan_chunk(d);
    if (!C) return false;
    const int64_t nchunks = (max_T + C - 1) / C;
    auto finish_packed = [&](int64_t segments, PrefillPlan *p) {
        finish_plan(d, C, segments, nchunks, false, p);
        if (p->segments == 1) return;
        const int D = d.d_k;
        auto up = [](size_t n) { return (n + 255) / 256 * 256; };
        p->max_pre_items = total_T / p->segment_tokens;
        p->max_items = p->max_pre_items + d.B;
        p->max_cut = p->max_pre_items < d.B ? p->max_pre_items : d.B;
        const size_t slots = static_cast<size_t>(p->max_items) * d.H;
        p->ws_state_bytes = slots * 2 * D * D * sizeof(float);
        p->ws_decay_bytes = up(slots * 2 * D * sizeof(float));
        p->ws_lists_bytes = lists_bytes(d, *p);
        p->ws_total_bytes = p->ws_ask_bytes = p->ws_need_bytes = p->ws_state_bytes + p->ws_decay_bytes + p->ws_lists_bytes;
    };
    int64_t P, P_cut;   // what is done; what the cut alone would be
    bool must_cut = true;
    double cut_cost = 0;   // of cutting every sequence, where that pays
    if (d.segments > 0) {
        P = P_cut = d.segments;
    } else {
        const int64_t target = (d.d_k == 64) ? 512 : 256;
        int64_t cps = (total_T * d.H / target + C - 1) / C;   // chunks per segment
        if (cps < 4) cps = 4;
        P = P_cut = (nchunks + cps - 1) / cps;
        if (P > 1) {
            const double chip = chip_slots(d), steps = static_cast<double>(total_T) / 32;
            const double L = static_cast<double>((nchunks + P - 1) / P * C);   // finish_plan evens the segments out
            const double n = L / 32, longest = static_cast<double>(max_T) / 32;
            const double cuts = static_cast<double>(total_T) / L * d.H, items = cuts + static_cast<double>(d.B) * d.H;
            auto costs = [&](const PrefillCosts &c) {   // whole, cut
                auto loop = [&](double chain, double workgroups) {
                    const double step = workgroups <= 256 ? c.step_alone : c.step;
                    const double spread = workgroups / chip * c.wg + steps * d.H / chip * c.step_full;
                    return spread > c.wg + chain * step ? spread : c.wg + chain * step;
                };
                const double whole = loop(longest, static_cast<double>(d.B) * d.H);
                return std::make_pair(whole, c.lists + c.wg + (cuts > chip ? cuts / chip : 1.0) * n * c.pre + c.slot * cuts + loop(n, items));
            };
            const auto before = costs(refusal_costs(d)), now = costs(prefill_costs(d));
            must_cut = before.first > before.second;
            if (now.first > now.second) cut_cost = now.second;
            else P = 1;
        }
    }
    finish_packed(P, plan);
    if (!must_cut && plan->ws_total_bytes > available) finish_packed(P = 1, plan);
    plan->longest_first = plan->segments == 1 && order_pays(d, total_T, max_T);
    if (P > 1 && cut_cost > 0 && plan->ws_total_bytes <= available)   // (its bytes are there: the long ones alone, if that is better still)
        cut_long(d, total_T, max_T, plan->ws_total_bytes, cut_cost, plan);
    if (P < P_cut) {
        // Whole by the estimate: the size query still answers with what cutting takes, if any smaller batch is cut, so that a
        // buffer sized for a large batch serves smaller ones.  The least a cut can cost is that of one sequence of n chunks.
        const PrefillCosts c = prefill_costs(d);
        bool some = nchunks > 64;
        for (int64_t n = 5; n <= nchunks && !some; ++n)
            for (int64_t most = 4; most < 8 && !some; ++most) {
                const int64_t tokens = n * C < max_T ? n * C : max_T, parts = (n + most - 1) / most;
                const double chain = static_cast<double>((n + parts - 1) / parts * C) / 32;
                some = parts > 1 && c.wg + static_cast<double>(tokens) / 32 * c.step > c.lists + 2 * c.wg + chain * (c.pre + c.step) + c.slot * d.H;
            }
        if (some) {
            PrefillPlan cut;
            finish_packed(P_cut, &cut);
            if (P == 1) cut_long(d, total_T, max_T, available < cut.ws_total_bytes ? available : cut.ws_total_bytes, 0, plan);
            plan->ws_ask_bytes = cut.ws_total_bytes;
        }
    }
    return true;
}

hipError_t launch_prefill(const dsla_desc &d, const PrefillPlan &plan, int64_t T, const int32_t *cu_seqlens,
                          const int32_t *seq_index, const int32_t *state_slot, const void *q, const void *k, const void *v, const void *g1,
                          const void *g2, float *S1, float *S2, void *o, void *workspace, hipStream_t stream,
                          const PrefillExt *ext)
{
    PrefillArgs a;
    a.slot_mul = 1;
    a.Hkv = ext ? ext->Hkv : d.H;
    a.explicit_w = ext ? 1 : 0;
    a.accumulate = ext ? ext->accumulate : 0;
    a.beta = ext ? ext->beta : 0;
    a.wa = ext ? ext->wa : 0.f;
    a.wb = ext ? ext->wb : 0.f;
    a.wa_per_head = ext ? ext->wa_per_head : nullptr;
    a.wb_per_head = ext ? ext->wb_per_head : nullptr;
    a.q = q; a.k = k; a.v = v; a.g1 = g1; a.g2 = g2; a.o = o;
    a.S1 = S1; a.S2 = S2;
    a.ws_state = static_cast<float *>(workspace);
    a.ws_decay = plan.segments > 1
                     ? reinterpret_cast<float *>(static_cast<char *>(workspace) + plan.ws_state_bytes)
                     : nullptr;
    a.gamma_per_head = d.gamma_per_head;
    a.cu = cu_seqlens;
    a.seq = seq_index;
    a.slot = state_slot;
    a.seg_first = a.seg_count = a.cut_seq = nullptr;
    a.list_full = a.list_pre = nullptr;
    if (plan.max_items > 0) {   // packed sequences, more than one segment: carve the work lists
        auto up = [](size_t n) { return (n + 255) / 256 * 256; };
        char *w = static_cast<char *>(workspace) + plan.ws_state_bytes + plan.ws_decay_bytes;
        a.seg_first = reinterpret_cast<int32_t *>(w);
        w += up((static_cast<size_t>(d.B) + 1) * 4);
        a.seg_count = reinterpret_cast<int32_t *>(w);
        a.cut_seq = a.seg_count + 4;
        w += up((static_cast<size_t>(d.B) + 4) * 4);
        a.list_full = reinterpret_cast<int4 *>(w);
        w += up(plan.max_items * 16);
        a.list_pre = reinterpret_cast<int4 *>(w);
    }
    a.longest_first = plan.longest_first ? 1 : 0;
    a.T = T;
    a.seg_tokens = plan.segment_tokens;
    a.H = d.H;
    a.P = plan.segments;
    a.zero_init = d.zero_init != 0;
    a.status = d.status;
    a.gamma = d.gamma;
    a.scale = d.scale;
    a.gate_inv_tau = d.gate_mode == DSLA_GATE_PREACT ? 1.0f / d.tau : 0.f;
    if (!ext && !cu_seqlens && !state_slot && prefill_short_built(d) && prefill_short_cost(d, T) < plan_cost(d, plan, T))
        return launch_prefill_short(d, a, stream);
    const int D = d.d_k;
    if (d.io_dtype == DSLA_BF16) {
        if (D == 128) return launch_g<128, bf16_t>(d, plan, a, stream);
        if (D == 64) return launch_g<64, bf16_t>(d, plan, a, stream);
    } else {
        if (D == 128) return launch_g<128, float>(d, plan, a, stream);
        if (D == 64) return launch_g<64, float>(d, plan, a, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace dsla
