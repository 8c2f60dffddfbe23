// What the prefill kernels share: their arguments, access to LDS by byte address, the map of gate pre-activations.
#pragma once
#include "dsla_internal.h"

namespace dsla {

struct PrefillArgs {
    const void *q, *k, *v, *g1, *g2;
    void *o;
    float *S1, *S2;          // caller's states
    // One workspace slot per (segment, sequence, head): slot = (p B + b) H + h, or with work lists as the entry says, times H, + h.
    // The last segment of a sequence has no decay entry that anyone reads.
    float *ws_state;         // [slot][2][D][D] fp32 (P > 1): state at the start of the segment
    float *ws_decay;         // [slot][2][D] fp32 (P > 1): log2 of the decay over the segment
    const float *gamma_per_head;
    const int32_t *cu;       // packed sequences: [B + 1] token offsets (sequence b = tokens cu[b] .. cu[b+1]-1); or null
    const int32_t *seq;      // with cu: [B] which of the packed sequences take part (entry b names sequence seq[b]); or null (all, in order)
    const int32_t *slot;     // [B] index of each sequence's states in S1, S2; or null (sequence b uses entry b)
    // Packed sequences of which any are cut: the work lists written by segment_list_kernel.  A workgroup is (list entry, head);
    // entries past the count exit.  An entry: sequence, first token, token past the last, slot of the state on entry
    // (-1: the sequence is whole).  Null when every sequence is one segment or cu is null.
    const int32_t *seg_first;   // [B + 1] first slot of each sequence (a sequence that is cut into n pieces by the pre-pass has n + 1)
    const int32_t *seg_count;   // [3] entries in list_full, list_pre, cut_seq
    const int32_t *cut_seq;     // the sequences that are cut
    const int4 *list_full;      // the chunk loop's segments
    const int4 *list_pre;       // the pre-pass's pieces: the segment, or a part of it, of every segment that is followed by another one
    int64_t T;               // tokens per sequence (cu == null); with cu: upper bound of the sequence lengths
    int64_t seg_tokens;
    int H;
    int P;
    int zero_init;           // nonzero: the states are zero on entry (the caller's S1, S2 are only written)
    int32_t *status;         // optional device word: set to DSLA_STATUS_GATE_DOMAIN by a step whose gates leave the domain
    float gamma, scale;
    // Extended launches (Kern<.., kExt = true>): explicit blend coefficients of the two states instead of
    // (gamma, 1 - gamma), key/value heads shared by groups of query heads, and output added to what o holds.
    int Hkv;                 // key/value heads (k, v are [..][Hkv][D]); == H in ordinary launches
    int explicit_w;          // nonzero: the blend coefficients are wa, wb (or the per-head arrays)
    int accumulate;          // nonzero: o += result instead of o = result
    int beta;                // nonzero (Kern<.., kBeta = true>): one state with the outer-product gate, see "Beta mode"
    float wa, wb;
    const float *wa_per_head, *wb_per_head;   // optional [H]
    float gate_inv_tau;      // 0: g1, g2 are log-gates; else they are pre-activations and this is 1 / tau
    int longest_first;       // chunk loop on whole packed sequences: workgroups take them in the order of their lengths
    int slot_mul;            // chunk loop: segment p starts from workspace slot p * slot_mul (the pre-pass and the scan may
                             // work on pieces of a segment: see PrefillPlan::pre_split)
};

// Short prompts in one launch (prefill_short.hip): whether it is built for a call, its estimate in us, and the launch.
bool prefill_short_built(const dsla_desc &d);
double prefill_short_cost(const dsla_desc &d, int64_t T);
hipError_t launch_prefill_short(const dsla_desc &d, const PrefillArgs &a, hipStream_t stream);

namespace {

constexpr float kLog2e = 1.4426950408889634f;

// Workgroup barrier that orders LDS traffic only.  __syncthreads() would also wait for the global
// loads of the next chunk that are deliberately left in flight across the contraction phases.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_sched_barrier(0);   // phases are not interleaved by the instruction scheduler
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------------------------
// LDS access by byte address.  Every LDS address below is "per-lane base register + compile-time
// constant"; the bases are computed once and passed through opaque() so that the compiler keeps them
// as they are instead of materialising one register per (base, constant) pair.
// ---------------------------------------------------------------------------------------------
#define DSLA_LDS __attribute__((address_space(3)))
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t lds_addr_of(const void *p)
{
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DSLA_LDS const char *)p));
}
__device__ __forceinline__ uint32_t opaque(uint32_t x)
{
    asm volatile("" : "+v"(x));
    return x;
}
template <class T>
struct LdsPtr {
    typedef T DSLA_LDS *type;   // pointer into LDS (32-bit)
};
template <class T>
__device__ __forceinline__ T lds_ld(uint32_t a)
{
    return *reinterpret_cast<typename LdsPtr<const T>::type>(static_cast<uintptr_t>(a));
}
template <class T>
__device__ __forceinline__ void lds_st(uint32_t a, T v)
{
    *reinterpret_cast<typename LdsPtr<T>::type>(static_cast<uintptr_t>(a)) = v;
}

// The largest exponent a step of 32 tokens may produce: its factors carry 2^{+-R/2}, and bf16 / fp32 hold 2^{+-126}.
constexpr float kMaxStepLog2Decay = 230.f;
// tau log2 alpha of a pre-activation
__device__ __forceinline__ float log2_sigmoid(float z)
{
    const float y = z * kLog2e;
    return fminf(y, 0.f) - __builtin_amdgcn_logf(1.0f + __builtin_amdgcn_exp2f(-__builtin_fabsf(y)));
}

}  // namespace
}  // namespace dsla
