// Causal softmax attention over a whole prompt: the prefill of a layer that has NOT been converted, which a partly
// converted model runs beside its DSLA layers (paper Section 4.3) and against which the linear-time DSLA prefill is
// measured (Section 5.3: quadratic against linear cost, crossing near 2K tokens).
//     o_t = sum_{i <= t} softmax_{i <= t}(scale * q_t . k_i) v_i
//
// One pass over the keys with a running reference maximum (the scores never leave the chip).  A workgroup of four
// wavefronts takes 128 consecutive queries of one (batch, head); a wavefront owns 32 of them.  Keys and values stream
// through LDS 64 at a time, shared by the four wavefronts, by buffer loads that go from memory straight to LDS (no
// staging registers, no LDS store instructions; see AttnTiles for the placement that keeps the reads conflict-free).
// Per block of 64 keys a wavefront computes two transposed score tiles S^T[key][query] = K Q^T on MFMA (so that a lane
// holds the scores of ONE query), with minus the query's reference as the initial accumulator, exponentiates, and adds
// V^T P^T to its output tiles O^T[column][query].
// The causal mask is applied only in the blocks on the diagonal, and the reference is raised (and the output tiles
// rescaled) only when a block exceeds it by more than 2^8, which after the first blocks is rare; the exchange between the
// two lanes of a query and the floating-point maximum exist only on that path.  Because an MFMA
// result tile and an MFMA input fragment both index lanes by the tile column, the exponentiated tile is fed back as
// the input fragment of the second product without passing through LDS; V sits in LDS as its rows arrived and its
// transposed fragments come from the transposing LDS read, in the key order the result registers of a score tile have.
//
// Bound by the matrix pipes and the power they draw: per wavefront and block 32 MFMAs (1024 cycles) against about 600 cycles of
// vector work and 320 of LDS transfers, with two wavefronts per SIMD to overlap them.  B = 8, H = 32, T = 8192, d = 128:
// 5.74 ms = 766 TFLOP/s before; heads kept on one XCD 4.44; a vector instruction per score less, LDS reads ahead of
// their MFMAs and exponentials under the MFMAs of the second product 3.92; loads the compiler does not wait for and a
// raised priority in the second product 3.79 ms = 1160 TFLOP/s (a plain library product of 8192^3: 1400).  Workgroups of eight
// wavefronts: 3.74 ms, but 54 against 47 us at B = 1, T = 2048 and 27 against 20 us at 24 heads of 1000 tokens.
// bf16 operands, fp32 accumulation and softmax statistics.  Short prompts of few heads have a kernel of their own (below).
#include "dsla_internal.h"

namespace dsla {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 4;                                 // wavefronts per workgroup
constexpr int kQueriesPerWg = 32 * kWaves;
constexpr int kKeys = 64;            // keys per block: two score tiles of 32
// The reference of a query is only raised when a block exceeds it by more than this (log2 units): the
// exponentials then stay below 2^8 and the output tiles are rescaled once in a long while instead of once per block.
// The normalisation at the end uses the same reference for numerator and denominator, so the result is the same sum.
constexpr float kMaxSlack = 8.0f;

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    f32x2 x = {a, b};
    bf16x2 y = __builtin_convertvector(x, bf16x2);
    return __builtin_bit_cast(uint32_t, y);
}
// LDS image of a block of 64 keys (and of its values): rows of d elements WITHOUT padding, because the block is
// written by loads that go from memory straight to LDS (a wavefront's 64 lanes fill 1 KB of consecutive LDS).  Bank
// conflicts are avoided by WHERE in its row a 16-byte piece is put:
// - keys: piece c of row r sits at piece position c ^ swz_k(r); the 16 rows that 16 lanes read at one time at the
//   same logical piece then fall into 16 different groups of four banks;
// - values: the 64-byte quarter q of row r sits at quarter position q ^ swz_v(r); a pass of the transposing read
//   takes one quarter from each of 4 consecutive rows, which then fall into the four quarters of the banks.
// The lane that fills LDS slot (row, position) simply fetches the piece that belongs there.
template <int D>
struct AttnTiles {
    static constexpr int RB = D * 2;                    // bytes per row
    static constexpr int NC = D / 8;                    // 16-byte pieces per row (16 or 8)
    static constexpr int NQ = RB / 64;                  // 64-byte quarters per row (4 or 2)
    static constexpr uint32_t K_BYTES = kKeys * RB;
    static constexpr uint32_t V_BYTES = kKeys * RB;
    static constexpr uint32_t BUF_BYTES = K_BYTES + V_BYTES;
    static __device__ __forceinline__ uint32_t swz_k(uint32_t row) { return NC == 16 ? (row & 15u) : ((row >> 1) & 7u); }
    static __device__ __forceinline__ uint32_t swz_v(uint32_t row) { return NQ == 4 ? (row & 3u) : ((row >> 1) & 1u); }
};

// Fragment of V^T for a block of 16 keys from V rows in LDS, by two transposing 8-byte reads: the 16 lanes of a group
// address 4 keys x 4 pieces of 4 columns and each receives 4 keys of ONE column.  With `a` as computed in the kernel
// lane l ends up with column (tile) + l % 32 and keys 4 g + 0..3 (from a) and 8 + 4 g + 0..3 (from a + 8 rows): the
// order in which the result registers of a score tile hold the keys.
__device__ __forceinline__ bf16x8 load_vt_frag(const char *a, uint32_t step)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef s16x4 __attribute__((address_space(3))) *lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(a));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(a + step));
    const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
    return __builtin_bit_cast(bf16x8, u32x4{l2[0], l2[1], h2[0], h2[1]});
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane from the buffer `res` at `voff` (per lane) into LDS at `lds` (uniform) + 16 * lane; the compiler does
// not know these loads: whoever reads the bytes waits with loads_landed_barrier() first.
__device__ __forceinline__ void load_to_lds16(const char *lds, uint32_t voff, u32x4 res)
{
    const uint32_t at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char *)lds));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(at), "v"(voff), "s"(res) : "m0", "memory");
}
#pragma clang diagnostic pop
__device__ __forceinline__ void loads_landed_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ u32x4 buffer_of(const void *p, int bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    return u32x4{static_cast<uint32_t>(a), static_cast<uint32_t>(a >> 32) & 0xffffu, static_cast<uint32_t>(bytes), 0x00020000u};
}

template <int D>
__global__ __launch_bounds__(64 * kWaves, 2) void attention_prefill_kernel(const bf16_t *__restrict__ q, const bf16_t *__restrict__ k,
                                                                   const bf16_t *__restrict__ v, bf16_t *__restrict__ o,
                                                                   int BH, int H, int T, int blocks_per_seq, float scale_log2e)
{
    using L = AttnTiles<D>;
    constexpr int NKB = D / 16;    // contraction blocks over the features
    constexpr int CT = D / 32;     // output column tiles
    __shared__ __attribute__((aligned(1024))) char buf_a[L::BUF_BYTES];
    __shared__ __attribute__((aligned(1024))) char buf_b[L::BUF_BYTES];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 31, g = lane >> 5;
    // Heads run fastest, in groups of kHeads: workgroup ids go round-robin over the 8 XCDs, so in a group of a multiple of
    // 8 heads a head stays on one XCD (of 12 or 28 heads on two, of an odd number on all), whose L2 serves its keys and
    // values to all query blocks that are in flight, and the heavy blocks (late queries: more keys) of the whole group come
    // first.  B = 8, H = 32, T = 8192: one head after the other over all XCDs 5.63 ms (every XCD reads the keys and values
    // of all heads in flight, 32 MB against 4 MB of L2); groups of 8, 16, 32, 64 heads 4.61, 4.42, 4.44, 4.54 ms.
    // T = 2048, B = 1: 70, 66, 65, 55, 55 us (with few heads an early end of the light blocks leaves the chip idle).  At
    // d = 64 a head has half the bytes.  (A single group does without the division by the size of the groups: an index
    // division is 0.05 of the 3.4 us of a call of one block of queries.)
    constexpr int kHeads = D == 128 ? 32 : 64;
    const int h0 = BH > kHeads ? static_cast<int>(blockIdx.x / (kHeads * blocks_per_seq)) * kHeads : 0;
    const int in_group = blockIdx.x - h0 * blocks_per_seq, heads = BH - h0 < kHeads ? BH - h0 : kHeads;
    const int bh = h0 + in_group % heads, qb = blocks_per_seq - 1 - in_group / heads;
    const int b = bh / H, h = bh % H;
    const int q0 = qb * kQueriesPerWg;
    const size_t rs = static_cast<size_t>(H) * D;                                   // elements between tokens
    const size_t base = (static_cast<size_t>(b) * T * H + h) * D;                   // (b, 0, h, 0)

    // ---- this lane's query: features 16 kb + 8 g .. + 7 for every kb, scaled by scale * log2 e, as bf16 ----
    const int wq0 = q0 + 32 * wave;   // first query of this wavefront
    const int my_q = wq0 + ln;
    const bool q_live = my_q < T;
    bf16x8 qf[NKB];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        u32x4 u = {0, 0, 0, 0};
        if (q_live) u = *reinterpret_cast<const u32x4 *>(q + base + static_cast<size_t>(my_q) * rs + 16 * kb + 8 * g);
        u32x4 s;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            s[w] = pack2(__uint_as_float(u[w] << 16) * scale_log2e, __uint_as_float(u[w] & 0xffff0000u) * scale_log2e);
        qf[kb] = __builtin_bit_cast(bf16x8, s);
    }

    // ---- staging of a key/value block: buffer loads with LDS as destination.  One instruction of a wavefront fills
    // 1 KB = RPI rows; instruction n = wave + kWaves i of a block fills rows n RPI .. of the keys (and one more of the
    // values).  The descriptors cover this (batch, head)'s keys and values from token 0 to the end of the last token's
    // row: rows past the end of the sequence arrive as zeros (they lie after every query and are masked). ----
    constexpr int RPI = 1024 / L::RB;                  // rows per instruction (4 or 8)
    constexpr int NI = kKeys / RPI / kWaves;           // instructions per wavefront, block and tensor
    static_assert(NI >= 1, "every wavefront stages something");
    const uint32_t rs2 = static_cast<uint32_t>(rs) * 2;   // bytes between tokens
    const int kv_bytes = static_cast<int>(static_cast<uint32_t>(T - 1) * rs2 + D * 2);   // an unsigned 32-bit count to the hardware
    const u32x4 res_k = buffer_of(k + base, kv_bytes), res_v = buffer_of(v + base, kv_bytes);
    const uint32_t uwave = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(wave));
    // this lane's LDS slot in an instruction: row lr of its RPI rows, piece position lp; the swizzles of the rows an
    // instruction fills depend on the lane and the wavefront only (RPI n is a multiple of what they look at)
    const uint32_t lr = static_cast<uint32_t>(lane) / L::NC, lp = static_cast<uint32_t>(lane) % L::NC;
    const uint32_t row0 = RPI * uwave + lr;            // row of instruction i = 0
    const uint32_t goff_k = lr * rs2 + 16 * (lp ^ L::swz_k(row0));
    const uint32_t goff_v = lr * rs2 + 16 * ((((lp >> 2) ^ L::swz_v(row0)) << 2) | (lp & 3u));
    auto stage_block = [&](char *buf, int key0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const uint32_t n = uwave + kWaves * i;
            // the range check is on the lane offset alone, so the row goes into it
            const uint32_t rowoff = (static_cast<uint32_t>(key0) + RPI * n) * rs2;
            load_to_lds16(buf + n * 1024, rowoff + goff_k, res_k);
            load_to_lds16(buf + L::K_BYTES + n * 1024, rowoff + goff_v, res_v);
        }
    };
    // fragment reads.  Keys: row 32 t + ln, logical piece 2 kb + g.  Values (transposing reads): the 16 lanes of a
    // group address 4 rows x 4 pieces of 4 columns: row 4 g + l16 / 4 of a block of 16 keys (+ 8 for the second read),
    // columns 32 ct + 16 (lane / 16 % 2) + 4 (l16 % 4), i.e. quarter ct of the row.
    const uint32_t sk = L::swz_k(ln);                  // (rows 32 t + ln: the swizzle looks at the low bits only)
    const uint32_t kf_off = ln * L::RB + 16 * ((g ^ sk) & 1u);
    const uint32_t kf_s1 = sk >> 1;                    // piece pair kb of the row sits at pair position kb ^ kf_s1
    const uint32_t l16 = lane & 15;
    const uint32_t vrow = 4 * g + (l16 >> 2);
    const uint32_t sv = L::swz_v(vrow);                // (rows 16 kb2 + 8 h + vrow: low bits only)
    const uint32_t vt_off = vrow * L::RB + 32 * ((lane >> 4) & 1) + 8 * (l16 & 3);

    // keys this workgroup needs: 0 .. min(T, q0 + 128) - 1; this wavefront needs them up to its last query
    const int wg_last_q = (q0 + kQueriesPerWg < T ? q0 + kQueriesPerWg : T) - 1;
    const int nblocks = wg_last_q / kKeys + 1;
    const int wave_last_q = wq0 + 31;

    f32x16 oacc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[ct][r] = 0.f;
    f32x16 mneg;   // minus the reference maximum (log2 domain) of this lane's query, in the shape of a score tile
#pragma unroll
    for (int r = 0; r < 16; ++r) mneg[r] = 0.f;
    float l_run = 0.f;   // this lane's share of the denominator (the other half of the keys is with lane + 32)

    auto compute = [&](const char *buf, int jb) {
        const int key0 = jb * kKeys;
        if (key0 <= wave_last_q) {   // else: every key of the block lies after every query of this wavefront
            const char *kb_ = buf;
            const char *vb_ = buf + L::K_BYTES;
            // S^T[key][query] - reference, two tiles of 32 keys: lane (ln, g) ends up with keys 32 t + 8 (r / 4) + 4 g + r % 4
            // of query ln.  Six fragments are on their way before the first MFMA, and the first values during the last.
            f32x16 sc[2];
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const bf16x8 kf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kb_ + 32 * t * L::RB + kf_off + 32 * (kb ^ kf_s1)));
                    sc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kb], kb ? sc[t] : mneg, 0, 0, 0);
                }
            bf16x8 vf[2][CT];
            auto read_v = [&](int s, int kb2) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) vf[s][ct] = load_vt_frag(vb_ + vt_off + 16 * kb2 * L::RB + 64 * (ct ^ sv), 8 * L::RB);
            };
            read_v(0, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
            for (int i = 0; i < 2 * NKB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (i < 2 * NKB - 6) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                else __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
            // causal mask, only in the blocks that reach past the first query of the wavefront (keys past the end of
            // the sequence lie after every query)
            if (key0 + kKeys - 1 > wq0) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = key0 + 32 * t + 8 * (r >> 2) + 4 * g + (r & 3);
                        sc[t][r] = key <= my_q ? sc[t][r] : -1.0e30f;
                    }
            }
            // Does any score exceed the reference by more than the slack, or has a query not seen a key yet?  (As signed
            // integers positive floats keep their order and lie above all negative ones: no canonicalisation.)
            int top = 0;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int x = __float_as_int(sc[t][r]);
                    top = top > x ? top : x;
                }
            if (__builtin_amdgcn_ballot_w64(top > __float_as_int(kMaxSlack) || l_run == 0.f) != 0) {
                float bmax = sc[0][0];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) bmax = fmaxf(bmax, sc[t][r]);
                bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
                const bool fresh = l_run + __shfl_xor(l_run, 32) == 0.f;   // nothing summed yet: any reference will do
                const float up = fresh ? (bmax > -1.0e30f ? bmax : 0.f) : fmaxf(bmax, 0.f);   // (-1e30: masked; -inf: no weight yet)
                const float alpha = fresh ? 1.f : __builtin_amdgcn_exp2f(-up);
                l_run *= alpha;
#pragma unroll
                for (int r = 0; r < 16; ++r) mneg[r] -= up;
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) sc[t][r] -= up;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int r = 0; r < 16; ++r) oacc[ct][r] *= alpha;
            }
            // 16 keys at a time: the exponentials, sums and packing of the next 16 and the reads of their values run under the
            // MFMAs of the current ones, which feed the halves of the score tiles back as input fragments
            float psum[2] = {0.f, 0.f};
            bf16x8 pf[2];
            auto exps = [&](int s, int kb2) {
                const f32x16 &x = sc[kb2 >> 1];
                const int o8 = 8 * (kb2 & 1);
                float e[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    e[i] = __builtin_amdgcn_exp2f(x[o8 + i]);
                    psum[i & 1] += e[i];
                }
                const u32x4 u = {pack2(e[0], e[1]), pack2(e[2], e[3]), pack2(e[4], e[5]), pack2(e[6], e[7])};
                pf[s] = __builtin_bit_cast(bf16x8, u);
            };
            exps(0, 0);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int kb2 = 0; kb2 < 4; ++kb2) {
                if (kb2 + 1 < 4) {
                    read_v((kb2 + 1) & 1, kb2 + 1);
                    exps((kb2 + 1) & 1, kb2 + 1);
                }
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    oacc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kb2 & 1][ct], pf[kb2 & 1], oacc[ct], 0, 0, 0);
                if (kb2 + 1 < 4) {
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                        __builtin_amdgcn_sched_group_barrier(0x400, 8 / CT, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 12 / CT, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_s_setprio(0);
            l_run += psum[0] + psum[1];
        }
    };
    // Block j lives in buffer j % 2; its loads are issued one iteration ahead, right after the barrier that frees the
    // buffer, and the barrier in front of its use waits for them (the loads of every wavefront must have landed).
    stage_block(buf_a, 0);
    for (int jb = 0; jb < nblocks; jb += 2) {
        loads_landed_barrier();   // block jb is in buffer a; every wavefront is done with block jb - 1
        if (jb + 1 < nblocks) stage_block(buf_b, (jb + 1) * kKeys);
        compute(buf_a, jb);
        if (jb + 1 < nblocks) {
            loads_landed_barrier();   // block jb + 1 is in buffer b; every wavefront is done with block jb
            if (jb + 2 < nblocks) stage_block(buf_a, (jb + 2) * kKeys);
            compute(buf_b, jb + 1);
        }
    }

    // ---- o[query][32 ct + 8 (r / 4) + 4 g + r % 4] = O^T / denominator ----
    const float l_all = l_run + __shfl_xor(l_run, 32);
    if (q_live) {
        const float inv = 1.0f / l_all;   // the query's own key is never masked
        bf16_t *op = o + base + static_cast<size_t>(my_q) * rs;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
                *reinterpret_cast<u32x2 *>(op + 32 * ct + 8 * rb + 4 * g) =
                    u32x2{pack2(oacc[ct][4 * rb] * inv, oacc[ct][4 * rb + 1] * inv),
                          pack2(oacc[ct][4 * rb + 2] * inv, oacc[ct][4 * rb + 3] * inv)};
    }
}


// ---------------------------------------------------------------------------------------------------------------
// Short prompts and few heads: the chain of key blocks of a workgroup is the call
// ---------------------------------------------------------------------------------------------------------------
// With few workgroups nothing overlaps the latencies of a block of keys (LDS, the dependent MFMAs, the test of the reference),
// and a workgroup's chain of blocks is the call: 1.1 us a block in the kernel above, of which 0.4 are MFMAs.  Here a
// workgroup has 64 queries, 16 to a wavefront, on 16 x 16 x 32 MFMAs: half of the work behind each of those latencies, twice as many
// workgroups, and less than one tile of queries wasted on a short prompt.  Where the chains are long and workgroups few (GROUPS = 2),
// four more wavefronts take every other block of keys, and the two groups' sums meet in LDS at the end, relative to the higher
// of their references.  Before / one group / two (us, d = 128): 32 heads of 100 tokens 6.3 / 5.1 / 6.6, of 400 10.7 / 8.8 / 9.7, of 1500
// 31.6 / 28.8 / 39.8; 8 heads of 1000 18.3 / 15.1 / 14.3, of 2000 31.9 / 26.5 / 23.8; d = 64: 32 heads of 362 7.1 / 5.5 / 6.1; 4 heads of
// 4000 38.6 / 28.4 / 23.3.  Not here: a ring of three or four blocks (15.0 and 15.6 against 12.4 us at 575 tokens: it is not the
// loads that are waited for), wavefronts of 48 queries in workgroups of eight for long prompts (LDS traffic falls by a third, 8 x 32
// heads of 8192 tokens 3.71 against 3.73 ms).
constexpr int kShortQueries = 64;   // queries per workgroup
template <int D, int GROUPS>
__global__ __launch_bounds__(256 * GROUPS, 2) void attention_prefill_short_kernel(
    const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v, bf16_t *__restrict__ o, int BH, int H, int T,
    int blocks_per_seq, float scale_log2e)
{
    using L = AttnTiles<D>;
    constexpr int NKB = D / 32;       // contraction blocks over the features
    constexpr int KT = kKeys / 16;    // score tiles along the keys
    constexpr int CT = D / 16;        // output column tiles
    __shared__ __attribute__((aligned(1024))) char ring[2 * GROUPS][L::BUF_BYTES];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int grp = wave >> 2, w4 = wave & 3, r = lane & 15, g = lane >> 4;
    const int bh = blockIdx.x % BH, qb = blocks_per_seq - 1 - static_cast<int>(blockIdx.x) / BH;   // late queries, which have more keys, first
    const int b = bh / H, h = bh % H;
    const int q0 = qb * kShortQueries, my_q = q0 + 16 * w4 + r;
    const size_t rs = static_cast<size_t>(H) * D;                                   // elements between tokens
    const size_t base = (static_cast<size_t>(b) * T * H + h) * D;                   // (b, 0, h, 0)

    // ---- staging, as in the kernel above: the four wavefronts of a group fill its blocks.  Keys as there; values with the
    // 32-byte piece p of row r at position p ^ swz (a pass of the transposing read takes one piece of 8 consecutive rows) ----
    auto swz_v = [](uint32_t row) { return D == 128 ? (row & 7u) : ((row >> 1) & 3u); };
    constexpr int RPI = 1024 / L::RB, NI = kKeys / RPI / 4;
    const uint32_t rs2 = static_cast<uint32_t>(rs) * 2;
    const int kv_bytes = static_cast<int>(static_cast<uint32_t>(T - 1) * rs2 + D * 2);   // an unsigned 32-bit count to the hardware
    const u32x4 res_k = buffer_of(k + base, kv_bytes), res_v = buffer_of(v + base, kv_bytes);
    const uint32_t uw4 = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(w4));
    const uint32_t row0 = RPI * uw4 + static_cast<uint32_t>(lane) / L::NC, lp = static_cast<uint32_t>(lane) % L::NC;
    const uint32_t goff_k = row0 * rs2 + 16 * (lp ^ L::swz_k(row0)), goff_v = row0 * rs2 + 16 * (lp ^ (swz_v(row0) << 1));
    auto stage_block = [&](char *buf, int key0) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const uint32_t n = uw4 + 4 * i, rowoff = (static_cast<uint32_t>(key0) + RPI * 4 * i) * rs2;   // (the swizzles do not see rows 4 RPI apart)
            load_to_lds16(buf + n * 1024, rowoff + goff_k, res_k);
            load_to_lds16(buf + L::K_BYTES + n * 1024, rowoff + goff_v, res_v);
        }
    };
    const int wg_last_q = (q0 + kShortQueries < T ? q0 + kShortQueries : T) - 1;
    const int nblocks = wg_last_q / kKeys + 1, rounds = (nblocks + GROUPS - 1) / GROUPS;
    if (grp < nblocks) stage_block(ring[grp], grp * kKeys);

    bf16x8 qf[NKB];   // this lane's query: features 32 kb + 8 g .., scaled by scale * log2 e, as bf16
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        u32x4 u = {0, 0, 0, 0};
        if (my_q < T) u = *reinterpret_cast<const u32x4 *>(q + base + static_cast<size_t>(my_q) * rs + 32 * kb + 8 * g);
        u32x4 s;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            s[w] = pack2(__uint_as_float(u[w] << 16) * scale_log2e, __uint_as_float(u[w] & 0xffff0000u) * scale_log2e);
        qf[kb] = __builtin_bit_cast(bf16x8, s);
    }
    const uint32_t sk = L::swz_k(r), kf_off = r * L::RB;                       // keys: row 16 t + r, logical piece 4 kb + g
    const uint32_t vrow = 4 * g + (r >> 2), sv = swz_v(vrow), vt_off = vrow * L::RB + 8 * (r & 3);   // values: rows 4 g + r / 4 of a tile, piece ct

    f32x4 oacc[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) oacc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 mneg = {0.f, 0.f, 0.f, 0.f};   // minus the reference of this lane's query
    float l_run = 0.f;

    auto compute = [&](const char *kb_, int key0) {
        const char *vb_ = kb_ + L::K_BYTES;
        f32x4 sc[KT];   // lane (r, g): keys 16 t + 4 g + e of query r
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const bf16x8 kf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(kb_ + 16 * t * L::RB + kf_off + 16 * ((4 * kb + g) ^ sk)));
                sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[kb], kb ? sc[t] : mneg, 0, 0, 0);
            }
        constexpr int NV = 2 * CT, VD = 4;   // value fragments of a block, fragments on their way
        bf16x8 vf[VD];
        auto read_v = [&](int s) {   // fragment s: keys 32 (s / CT) .., columns 16 (s % CT) ..
            vf[s % VD] = load_vt_frag(vb_ + vt_off + 32 * (s / CT) * L::RB + 32 * ((s % CT) ^ sv), 16 * L::RB);
        };
#pragma unroll
        for (int s = 0; s < VD; ++s) read_v(s);
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
        for (int i = 0; i < KT * NKB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (i < KT * NKB - 6) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            else if (i < KT * NKB - 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        if (key0 + kKeys - 1 > q0 + 16 * w4) {   // reaches past the first query of the wavefront
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) sc[t][e] = key0 + 16 * t + 4 * g + e <= my_q ? sc[t][e] : -1.0e30f;
        }
        int top = 0;   // (as signed integers: see above)
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int x = __float_as_int(sc[t][e]);
                top = top > x ? top : x;
            }
        if (__builtin_amdgcn_ballot_w64(top > __float_as_int(kMaxSlack) || l_run == 0.f) != 0) {
            float bmax = sc[0][0];
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) bmax = fmaxf(bmax, sc[t][e]);
            bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
            bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
            float l_all = l_run + __shfl_xor(l_run, 16);
            l_all += __shfl_xor(l_all, 32);
            const bool fresh = l_all == 0.f;   // nothing summed yet: any reference will do
            const float up = fresh ? (bmax > -1.0e30f ? bmax : 0.f) : fmaxf(bmax, 0.f);   // (-1e30: masked; -inf: no weight yet)
            const float alpha = fresh ? 1.f : __builtin_amdgcn_exp2f(-up);
            l_run *= alpha;
#pragma unroll
            for (int e = 0; e < 4; ++e) mneg[e] -= up;
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) sc[t][e] -= up;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int e = 0; e < 4; ++e) oacc[ct][e] *= alpha;
        }
        // 32 keys at a time (two score tiles are an input fragment): the exponentials of the second 32 run under the MFMAs of the
        // first, and the values are read four fragments ahead
        bf16x8 pf[2];
        auto exps = [&](int half) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = __builtin_amdgcn_exp2f(sc[2 * half + (i >> 2)][i & 3]);
            l_run += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
            pf[half] = __builtin_bit_cast(bf16x8, u32x4{pack2(x[0], x[1]), pack2(x[2], x[3]), pack2(x[4], x[5]), pack2(x[6], x[7])});
        };
        exps(0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (half == 0) exps(1);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const int s = half * CT + ct;
                oacc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[s % VD], pf[half], oacc[ct], 0, 0, 0);
                if (s + VD < NV) read_v(s + VD);
            }
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (half * CT + ct + VD < NV) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                if (half == 0) {
                    __builtin_amdgcn_sched_group_barrier(0x400, 8 / CT, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 12 / CT, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    // round j: block GROUPS j + grp, loaded one round ahead into the other of the group's two buffers
    auto round = [&](int j, char *cur, char *nxt) {
        const int jb = GROUPS * j + grp;
        loads_landed_barrier();   // this round's blocks are there; everybody is done with the last round's
        if (jb + GROUPS < nblocks) stage_block(nxt, (jb + GROUPS) * kKeys);
        if (jb < nblocks && jb * kKeys <= q0 + 16 * w4 + 15) compute(cur, jb * kKeys);
    };
    char *const even = GROUPS == 1 ? ring[0] : ring[grp], *const odd = GROUPS == 1 ? ring[1] : ring[2 + grp];
    for (int j = 0; j < rounds; j += 2) {
        round(j, even, odd);
        if (j + 1 < rounds) round(j + 1, odd, even);
    }

    // ---- the second group's record goes through LDS to the first: its reference, denominator and sums per query ----
    float l_all = l_run + __shfl_xor(l_run, 16);
    l_all += __shfl_xor(l_all, 32);
    float f0 = 1.f, f1 = 0.f, l1 = 0.f;
    // per wavefront of a group: [CT][64] f32x4, then 64 x (reference, denominator)
    float *rec = reinterpret_cast<float *>(&ring[0][0]) + w4 * (CT * 256 + 128);
    if constexpr (GROUPS == 2) {
        __syncthreads();   // the last blocks have been read
        if (grp == 1) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) *reinterpret_cast<f32x4 *>(rec + ct * 256 + 4 * lane) = oacc[ct];
            rec[CT * 256 + 2 * lane] = mneg[0];
            rec[CT * 256 + 2 * lane + 1] = l_all;
        }
        __syncthreads();
        if (grp == 1) return;
        const float m1 = rec[CT * 256 + 2 * lane];
        l1 = rec[CT * 256 + 2 * lane + 1];
        // minus the references: the smaller one is the higher level.  A group without any weight (no key yet) does not count.
        const float low = l1 == 0.f ? mneg[0] : (l_all == 0.f ? m1 : fminf(mneg[0], m1));
        f0 = l_all == 0.f ? 0.f : __builtin_amdgcn_exp2f(low - mneg[0]);
        f1 = l1 == 0.f ? 0.f : __builtin_amdgcn_exp2f(low - m1);
    }
    if (my_q < T) {
        const float inv = 1.0f / (GROUPS == 2 ? f0 * l_all + f1 * l1 : l_all);   // the query's own key is never masked
        bf16_t *op = o + base + static_cast<size_t>(my_q) * rs;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            f32x4 x = oacc[ct];
            if constexpr (GROUPS == 2) {   // (a group that does not count may hold 0 times infinity)
                const f32x4 y = *reinterpret_cast<const f32x4 *>(rec + ct * 256 + 4 * lane);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = f1 == 0.f ? f0 * x[e] : (f0 == 0.f ? f1 * y[e] : f0 * x[e] + f1 * y[e]);
            }
            *reinterpret_cast<u32x2 *>(op + 16 * ct + 4 * g) = u32x2{pack2(x[0] * inv, x[1] * inv), pack2(x[2] * inv, x[3] * inv)};
        }
    }
}

// How many workgroups of 64 queries the kernel for short prompts still pays with; two (d = 64: four) are resident on a compute unit.
// Past that a second round of them costs what their shorter chains save, unless the chains are long (they even out) or a single
// block.  Before that the heads decide: those of a multiple of 8 stay on one XCD each, of 4 on two; of other numbers every XCD's L2 reads
// the keys of all heads, twice as often as with workgroups of 128 queries.  Before / now (us or, alone, now in parts of before),
// d = 128: 596 workgroups of 2 blocks 7.9 / 10.8, 756 of 4 (189 heads) 12.2 / 17.2, 512 (128 heads) 0.91, 376 of 8 (47 heads) 1.08, 544 (68 heads) 0.76, 640
// (80 heads) 0.90, 689 of 13 (53 heads) 1.16, 684 of 9 (76 heads) 0.89, 720 of 18 (40 heads) 0.75, 650 of 50 0.89; d = 64: 1014 of 2 1.03, 906 of
// 3 0.90, 756 of 4 (189 heads) 0.94, 836 (209 heads) 1.13, 1146 of 6 (191 heads) 11.7 / 15.8, 1176 of 7 (168 heads) 0.89, 1177 of 11 (107
// heads) 1.20, 1274 of 98 0.92.
int64_t most_short_workgroups(int d, int64_t heads, int64_t key_blocks)
{
    const bool wide = d == 128;
    if (key_blocks == 1 || key_blocks >= 20) return wide ? 768 : 1280;
    if (key_blocks <= 3) return wide ? 512 : (key_blocks == 2 ? 768 : 1024);
    if (heads % 4 == 0) {
        if (!wide) return 1088;
        if (heads % 8 == 0) return key_blocks == 4 ? 608 : 768;
        return key_blocks <= 6 ? 416 : (key_blocks <= 8 ? 560 : 768);
    }
    if (wide) return key_blocks <= 8 ? 288 : (key_blocks <= 12 ? 320 : 512);
    return key_blocks <= 5 ? 720 : (key_blocks <= 12 ? 640 : 768);
}

}  // namespace

hipError_t launch_attn_prefill(int B, int H, int d, int64_t T, float scale, const void *q, const void *k, const void *v,
                               void *o, hipStream_t stream)
{
    const float sl2 = scale * 1.4426950408889634f;
    ProfileScope ps(DSLA_KERNEL_ATTENTION_PREFILL, stream);
    const int64_t short_grid = static_cast<int64_t>(B) * H * ((T + kShortQueries - 1) / kShortQueries);
    const int64_t key_blocks = (T + kKeys - 1) / kKeys;
    if (short_grid <= most_short_workgroups(d, static_cast<int64_t>(B) * H, key_blocks)) {
        // Two groups where the chain has 16 blocks and every workgroup a compute unit to itself, or 32 blocks and two units' worth
        // of workgroups.  One / two groups: 128 workgroups, 16 blocks 15.1 / 14.3, 384, 16 blocks 18.4 / 18.7, 504, 63 blocks 56.3 / 49.6, 752, 47 30.2 / 29.9.
        const bool two = (short_grid <= 256 && key_blocks >= 16) || (short_grid <= 512 && key_blocks >= 32);
        auto launch = [&](auto kernel, int groups) {
            DSLA_LAUNCH(ps, kernel, dim3(static_cast<unsigned>(short_grid)), dim3(256 * groups), 0, stream, static_cast<const bf16_t *>(q),
                        static_cast<const bf16_t *>(k), static_cast<const bf16_t *>(v), static_cast<bf16_t *>(o), B * H, H, static_cast<int>(T),
                        static_cast<int>(short_grid / (static_cast<int64_t>(B) * H)), sl2);
        };
        if (two) launch(d == 128 ? attention_prefill_short_kernel<128, 2> : attention_prefill_short_kernel<64, 2>, 2);
        else launch(d == 128 ? attention_prefill_short_kernel<128, 1> : attention_prefill_short_kernel<64, 1>, 1);
        return hipGetLastError();
    }
    const int blocks_per_seq = static_cast<int>((T + kQueriesPerWg - 1) / kQueriesPerWg);
    const unsigned grid = static_cast<unsigned>(B) * H * blocks_per_seq;
    if (d == 128)
        DSLA_LAUNCH(ps, (attention_prefill_kernel<128>), dim3(grid), dim3(64 * kWaves), 0, stream, static_cast<const bf16_t *>(q),
                           static_cast<const bf16_t *>(k), static_cast<const bf16_t *>(v), static_cast<bf16_t *>(o), B * H, H,
                           static_cast<int>(T), blocks_per_seq, sl2);
    else
        DSLA_LAUNCH(ps, (attention_prefill_kernel<64>), dim3(grid), dim3(64 * kWaves), 0, stream, static_cast<const bf16_t *>(q),
                           static_cast<const bf16_t *>(k), static_cast<const bf16_t *>(v), static_cast<bf16_t *>(o), B * H, H,
                           static_cast<int>(T), blocks_per_seq, sl2);
    return hipGetLastError();
}

}  // namespace dsla
