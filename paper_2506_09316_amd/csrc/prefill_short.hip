// Short prompts, in the attention form of the layer: one launch, no workspace, no chain of steps.
//
// The step loop of prefill.hip walks a sequence 32 tokens at a time, and cutting it into segments adds a pre-pass and a scan: for
// a few hundred tokens the chain of steps, or the three launches, are the call.  Unrolled over the whole sequence (Section 4.1)
// the layer is causal attention without a softmax,
//     o_t = sum_{s <= t} [ sum_i gamma_i sum_f q_t[f] k_s[f] 2^{b^i_t[f] - b^i_s[f]} ] v_s          (b: running sums of log2 alpha)
//     S^i = sum_s (k_s 2^{b^i_T - b^i_s})^T v_s
// and every 16 queries, and every slice of a state, can be computed on their own.  That is quadratic in T, but nothing waits for
// anything: a workgroup is
//  * 16 queries of one head against all keys up to them: its wavefronts take 16 keys each, as many tiles at a time as there are
//    wavefronts, going back from the queries; partial outputs meet in LDS; or
//  * 32 columns of one state: its wavefronts take 16 tokens each of the update, going back from the end.
// Exponents are suffix sums from a tile to the queries (or the end): never positive, so nothing overflows whatever the gates,
// except inside the tile of the queries themselves, whose exponents are centred as those of a step are.  A lane prepares the 16
// tokens of a feature, so sums along a tile are plain additions and rows are loaded whole; sums over the tiles in between cross the
// wavefronts through LDS (two barriers per round), operands turn from features to tokens through the LDS of their wavefront, and the
// scores, whose lanes are queries, are fed to the product with V as they are.
//
// Bound by latency while the workgroups are few (one waits for its rows once, then for 6144 cycles of MFMAs at 16 tiles, d = 64), by
// the fp32 matrix pipe when they are many: n tiles are n (n + 1) / 2 pairs of 1536 (d = 64) or 3072 cycles per head, so the step
// loop is ahead again for long prompts and many heads (prefill_short_cost).  Step loop / this, us: d = 64, 4 heads of 64, 256, 512 tokens
// 11.2 / 6.3, 22.5 / 10.5, 47 / 17.0; d = 128, 8 heads 26.7 / 8.4, 47.4 / 18.2, 124 / 32.0; 32 heads of 64 and 256 27.3 / 14.9, 53.0 / 38.6.
// A lane that holds 16 features of one token, so that nothing turns through LDS, sums along a tile with DPP additions, five
// instructions per gate: 256 tokens, 4 heads 18.9.
#include "prefill_common.h"

namespace dsla {
namespace {

// The LDS pipeline takes the requests of one wavefront in order: only the compiler has to keep it.
__device__ __forceinline__ void wave_sync() { asm volatile("" ::: "memory"); }

template <int D, class TG, bool kPreact>
struct Short {
    static constexpr int NW = D == 64 ? 16 : 8, NT = 64 * NW, TT = 16;   // wavefronts (what registers and LDS hold); tokens per tile
    static constexpr int NH = D / 64;       // preparing: lane l has features l, l + 64
    static constexpr int NB = D / 16;       // multiplying: lane (r, g) has features 16 b + 4 g + i of row r; tiles of 16 columns or features
    static constexpr int SC = 32;           // columns of a state per workgroup
    static constexpr int RP = D + 4, QP = 2 * D + 4;            // row pitches (floats): a row shifts the banks by 16 bytes
    static constexpr uint32_t O_TOT = NW * TT * RP * 4;         // (first: the wavefronts' operands, later their sums) float [NW][2][D]: gate sums of the tiles, then their exponents
    static constexpr uint32_t O_Q = O_TOT + NW * 2 * D * 4;     // the queries' factors, from the start of their tile and centred on it
    static constexpr uint32_t Q_BYTES = TT * QP * 4;
    static constexpr uint32_t LDS_BYTES = O_Q + 2 * Q_BYTES;

    struct Place {
        int lane, r, g, w;   // lane (r, g), wavefront
        uint32_t sm, own;    // LDS, and the wavefront's part of it
        float unit;          // gate sums times this = log2 of a decay
        int64_t T;
        size_t base;         // element of the head's first token
        uint32_t rs;         // elements between tokens
    };
    static __device__ __forceinline__ int tokens_of(const Place &p, int j)   // of tile j, at least one
    {
        const int64_t left = p.T - static_cast<int64_t>(j) * TT;
        return left < TT ? static_cast<int>(left) : TT;
    }
    // 16 tokens of a tile's feature, the last token for those past the end
    template <class T>
    static __device__ __forceinline__ void load_column(T (&x)[TT], const T *tile, const Place &p, int n)
    {
#pragma unroll
        for (int t = 0; t < TT; ++t) x[t] = (tile + static_cast<size_t>(t < n ? t : n - 1) * p.rs)[p.lane];
    }
    static __device__ __forceinline__ void gates(float (&x)[TT], const TG (&g)[TT], int n)   // a token past the end: no decay
    {
#pragma unroll
        for (int t = 0; t < TT; ++t) x[t] = t < n ? (kPreact ? log2_sigmoid(to_f32(g[t])) : to_f32(g[t])) : 0.f;
    }
    // V[4 g + e][16 c + r]
    template <int C>
    static __device__ __forceinline__ void load_v(float (&v)[C][4], const float *tile, const Place &p, int n)
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = 4 * p.g + e;
            const float *row = tile + static_cast<uint32_t>(t < n ? t : n - 1) * p.rs + p.r;
#pragma unroll
            for (int c = 0; c < C; ++c) v[c][e] = row[16 * c];
        }
    }
    template <int C>
    static __device__ __forceinline__ void clear_v(float (&v)[C][4], const Place &p, int n)   // past the end
    {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < C; ++c) v[c][e] = 4 * p.g + e < n ? v[c][e] : 0.f;
    }
    // Sums over the later tokens of a tile, this token's own gate not among them; returns the sum over the tile
    static __device__ __forceinline__ float suffix_sums(float (&x)[TT])   // (in place)
    {
        float run = 0.f;
#pragma unroll
        for (int t = TT - 1; t >= 0; --t) {
            const float own = x[t];
            x[t] = run;
            run += own;
        }
        return run;
    }
    // Sums up to and including each token, from the middle of the tile's own total: the exponents of its queries, negated those of its
    // keys.  The same sums on both sides, and counted from the nearer end of the tile: one rounding at the size of the total, which a
    // single strong gate makes large for all tokens (one after the other from the middle: twice the error of the outputs).
    static __device__ __forceinline__ void centred_sums(const float (&x)[TT], float (&b)[TT])
    {
        float run = 0.f;
#pragma unroll
        for (int t = 0; t < TT; ++t) b[t] = run += x[t];
        const float half = 0.5f * run;
        float later = 0.f;
#pragma unroll
        for (int t = TT - 1; t >= 0; --t) {
            b[t] = b[t] > later ? b[t] - half : half - later;
            later += x[t];
        }
    }
    // keys times their decays -> LDS rows of the wavefront
    static __device__ __forceinline__ void store_keys(const Place &p, const float (&k)[TT], const float (&E)[TT], float off, int n, int hf)
    {
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            const float x = t < n ? k[t] * __builtin_amdgcn_exp2f(fmaf(E[t], p.unit, off)) : 0.f;
            lds_st<float>(p.own + (t * RP + 64 * hf + p.lane) * 4, x);
        }
    }
    static __device__ __forceinline__ f32x4 mma(float x, float y, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0); }

    // 16 queries (tile u) of a head
    static __device__ __forceinline__ void queries(const PrefillArgs &a, const Place &p, int u, int h)
    {
        const int rounds = u / NW + 1;
        const float *qp = static_cast<const float *>(a.q) + p.base, *kp = static_cast<const float *>(a.k) + p.base,
                    *vp = static_cast<const float *>(a.v) + p.base;
        const TG *gp[2] = {static_cast<const TG *>(a.g1) + p.base, static_cast<const TG *>(a.g2) + p.base};
        const uint32_t tot = p.sm + O_TOT + p.w * 2 * D * 4;
        f32x4 O[NB];   // [column 16 c + 4 g + e][query r]
#pragma unroll
        for (int c = 0; c < NB; ++c) O[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (NW - 1 - p.w < 2 * NH) {   // the queries' factors: a wavefront (of those that have the fewest keys) per state and 64 features
            const int s = (NW - 1 - p.w) / NH, hf = (NW - 1 - p.w) % NH, n = tokens_of(p, u);
            const size_t at = static_cast<size_t>(u) * TT * p.rs + 64 * hf;
            float q[TT], x[TT], b[TT], run = 0.f;
            TG g[TT];
            load_column(g, (s ? gp[1] : gp[0]) + at, p, n);
            load_column(q, qp + at, p, n);
            const float gm = a.gamma_per_head ? a.gamma_per_head[h] : a.gamma, gs = (s ? 1.0f - gm : gm) * a.scale;
            gates(x, g, n);
            centred_sums(x, b);
            const uint32_t row = p.sm + O_Q + (s * D + 64 * hf + p.lane) * 4;
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                run += x[t];
                q[t] *= gs;
                lds_st<float>(row + t * QP * 4, q[t] * __builtin_amdgcn_exp2f(p.unit * run));
                lds_st<float>(row + Q_BYTES + t * QP * 4, q[t] * __builtin_amdgcn_exp2f(p.unit * b[t]));
            }
        }
        float run = 0.f;   // of this thread's column (state, feature): gate sum of the tiles so far, without that of the queries
        for (int rd = 0; rd < rounds; ++rd) {
            const int j = u - rd * NW - p.w;
            const bool act = j >= 0;
            float k[NH][TT], E[2][NH][TT], v[NB][4];
            int n = 0;
            if (act) {
                n = tokens_of(p, j);
                const size_t at = static_cast<size_t>(j) * TT * p.rs;
                TG g[2][NH][TT];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int hf = 0; hf < NH; ++hf) load_column(g[s][hf], gp[s] + at + 64 * hf, p, n);
#pragma unroll
                for (int hf = 0; hf < NH; ++hf) load_column(k[hf], kp + at + 64 * hf, p, n);
                load_v(v, vp + at, p, n);
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int hf = 0; hf < NH; ++hf) {
                        float sum = 0.f;   // (the queries' own tile: none; its exponents are complete)
                        gates(E[s][hf], g[s][hf], n);
                        if (j < u) {
                            sum = suffix_sums(E[s][hf]);
                        } else {
                            float b[TT];
                            centred_sums(E[s][hf], b);
#pragma unroll
                            for (int t = 0; t < TT; ++t) E[s][hf][t] = -b[t];
                        }
                        lds_st<float>(tot + (s * D + 64 * hf + p.lane) * 4, sum);
                    }
            }
            lds_barrier();
            if (threadIdx.x < 2 * D) {   // the exponent of each tile: the sum of the tiles between it and the queries'
                const uint32_t col = p.sm + O_TOT + threadIdx.x * 4;
                float t[NW];   // (what lies past the first tile is not used)
#pragma unroll
                for (int i = 0; i < NW; ++i) t[i] = lds_ld<float>(col + i * 2 * D * 4);
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    lds_st<float>(col + i * 2 * D * 4, p.unit * run);
                    run += t[i];
                }
            }
            lds_barrier();
            if (act) {
                const bool diag = j == u;
                f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};   // [key 4 g + e][query r]
                const uint32_t qa = p.sm + O_Q + (diag ? Q_BYTES : 0) + (p.r * QP + 4 * p.g) * 4, ka = p.own + (p.r * RP + 4 * p.g) * 4;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
#pragma unroll
                    for (int hf = 0; hf < NH; ++hf) store_keys(p, k[hf], E[s][hf], lds_ld<float>(tot + (s * D + 64 * hf + p.lane) * 4), n, hf);
                    wave_sync();
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const f32x4 kf = lds_ld<f32x4>(ka + 64 * b), qf = lds_ld<f32x4>(qa + (s * D + 16 * b) * 4);
#pragma unroll
                        for (int i = 0; i < 4; ++i) sc[i & 1] = mma(kf[i], qf[i], sc[i & 1]);
                    }
                    wave_sync();
                }
                if (n < TT) clear_v(v, p, n);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = sc[0][e] + sc[1][e], P = !diag || 4 * p.g + e <= p.r ? x : 0.f;
#pragma unroll
                    for (int c = 0; c < NB; ++c) O[c] = mma(v[c][e], P, O[c]);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NB; ++c) lds_st<f32x4>(p.own + (p.r * RP + 16 * c + 4 * p.g) * 4, O[c]);
        lds_barrier();
        const int t = threadIdx.x / (D / 4), c4 = threadIdx.x % (D / 4) * 4;
        if (t < tokens_of(p, u)) {
            f32x4 sum = lds_ld<f32x4>(p.sm + (t * RP + c4) * 4);
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += lds_ld<f32x4>(p.sm + ((w * TT + t) * RP + c4) * 4);
            *reinterpret_cast<f32x4 *>(static_cast<float *>(a.o) + p.base + (static_cast<size_t>(u) * TT + t) * p.rs + c4) = sum;
        }
    }

    // columns 32 cg .. of state s of a head
    static __device__ __forceinline__ void state(const PrefillArgs &a, const Place &p, int ntiles, int s, int cg, size_t state0)
    {
        const float *kp = static_cast<const float *>(a.k) + p.base, *vp = static_cast<const float *>(a.v) + p.base + SC * cg;
        const TG *gp = static_cast<const TG *>(s ? a.g2 : a.g1) + p.base;
        const uint32_t tot = p.sm + O_TOT + p.w * 2 * D * 4;
        constexpr int C2 = SC / 16;
        f32x4 U[NB][C2];   // [feature 16 f + 4 g + e][column 16 c + r]
#pragma unroll
        for (int f = 0; f < NB; ++f)
#pragma unroll
            for (int c = 0; c < C2; ++c) U[f][c] = f32x4{0.f, 0.f, 0.f, 0.f};
        float run = 0.f, pair = 0.f;   // of this thread's feature: gate sum of the tiles so far; of the later half of a step
        const int rounds = (ntiles + NW - 1) / NW;
        for (int rd = 0; rd < rounds; ++rd) {
            const int j = ntiles - 1 - rd * NW - p.w;
            const bool act = j >= 0;
            float k[NH][TT], E[NH][TT], v[C2][4];
            int n = 0;
            if (act) {
                n = tokens_of(p, j);
                const size_t at = static_cast<size_t>(j) * TT * p.rs;
                TG g[NH][TT];
#pragma unroll
                for (int hf = 0; hf < NH; ++hf) load_column(g[hf], gp + at + 64 * hf, p, n);
#pragma unroll
                for (int hf = 0; hf < NH; ++hf) load_column(k[hf], kp + at + 64 * hf, p, n);
                load_v(v, vp + at, p, n);
#pragma unroll
                for (int hf = 0; hf < NH; ++hf) {
                    gates(E[hf], g[hf], n);
                    lds_st<float>(tot + (64 * hf + p.lane) * 4, suffix_sums(E[hf]));
                }
            }
            lds_barrier();
            if (threadIdx.x < D) {
                const uint32_t col = p.sm + O_TOT + threadIdx.x * 4;
                float t[NW];
#pragma unroll
                for (int i = 0; i < NW; ++i) t[i] = lds_ld<float>(col + i * 2 * D * 4);
#pragma unroll
                for (int i = 0; i < NW; ++i) {
                    lds_st<float>(col + i * 2 * D * 4, p.unit * run);
                    run += t[i];
                    pair += t[i];
                    const int tile = ntiles - 1 - rd * NW - i;
                    if ((tile & 1) == 0) {   // the first tile of a step of 32 tokens
                        if (tile >= 0 && a.status && cg == 0 && !(pair * p.unit >= -kMaxStepLog2Decay)) *a.status = DSLA_STATUS_GATE_DOMAIN;
                        pair = 0.f;
                    }
                }
            }
            lds_barrier();
            if (act) {
#pragma unroll
                for (int hf = 0; hf < NH; ++hf) store_keys(p, k[hf], E[hf], lds_ld<float>(tot + (64 * hf + p.lane) * 4), n, hf);
                wave_sync();
                if (n < TT) clear_v(v, p, n);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int f = 0; f < NB; ++f) {
                        const float x = lds_ld<float>(p.own + ((4 * p.g + e) * RP + 16 * f + p.r) * 4);
#pragma unroll
                        for (int c = 0; c < C2; ++c) U[f][c] = mma(x, v[c][e], U[f][c]);
                    }
                wave_sync();
            }
        }
        float *S = (s ? a.S2 : a.S1) + state0 + SC * cg;
        const int col = threadIdx.x & 15, f4 = threadIdx.x / 16 * 4;
#pragma unroll
        for (int c = 0; c < C2; ++c) {
            if (c) lds_barrier();
#pragma unroll
            for (int f = 0; f < NB; ++f) lds_st<f32x4>(p.own + (p.r * RP + 16 * f + 4 * p.g) * 4, U[f][c]);
            lds_barrier();
            if (f4 < D) {
                f32x4 sum = lds_ld<f32x4>(p.sm + (col * RP + f4) * 4);
#pragma unroll
                for (int w = 1; w < NW; ++w) sum += lds_ld<f32x4>(p.sm + ((w * TT + col) * RP + f4) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) S[(f4 + e) * D + 16 * c + col] = sum[e];
            }
        }
    }
};

// The states' workgroups (longest, so they come first), then the queries', the last ones of all heads first.
template <int D, class TG, bool kPreact>
__global__ __launch_bounds__((Short<D, TG, kPreact>::NT), (D == 64 ? 4 : 2)) void prefill_short_kernel(PrefillArgs a, int BH, int ntiles)
{
    using K = Short<D, TG, kPreact>;
    __shared__ __align__(16) unsigned char lds[K::LDS_BYTES];
    typename K::Place p;
    p.lane = threadIdx.x & 63;
    p.r = p.lane & 15;
    p.g = p.lane >> 4;
    p.w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    p.sm = lds_addr_of(lds);
    p.own = p.sm + p.w * K::TT * K::RP * 4;
    p.unit = kPreact ? a.gate_inv_tau : kLog2e;
    p.T = a.T;
    p.rs = static_cast<uint32_t>(a.H) * D;
    const int id = static_cast<int>(blockIdx.x), per_head = 2 * (D / K::SC), states = BH * per_head;
    const bool is_state = id < states;
    const int bh = (is_state ? id : id - states) % BH, part = (is_state ? id : id - states) / BH;
    p.base = (static_cast<size_t>(bh / a.H) * a.T * a.H + bh % a.H) * D;
    if (is_state) K::state(a, p, ntiles, part & 1, part >> 1, static_cast<size_t>(bh) * D * D);
    else K::queries(a, p, ntiles - 1 - part, bh % a.H);
}

template <int D, class TG>
hipError_t launch(const PrefillArgs &a, int B, hipStream_t stream)
{
    const int BH = B * a.H, ntiles = static_cast<int>((a.T + 15) / 16), states = BH * 2 * (D / 32), queries = BH * ntiles;
    ProfileScope ps(DSLA_KERNEL_PREFILL_CHUNK_LOOP, stream);
    if (a.gate_inv_tau != 0.f)
        DSLA_LAUNCH(ps, (prefill_short_kernel<D, TG, true>), dim3(states + queries), dim3(Short<D, TG, true>::NT), 0, stream, a, BH, ntiles);
    else
        DSLA_LAUNCH(ps, (prefill_short_kernel<D, TG, false>), dim3(states + queries), dim3(Short<D, TG, false>::NT), 0, stream, a, BH, ntiles);
    return hipGetLastError();
}

}  // namespace

// Calls that this is built for: one launch cannot read the states on entry, which it would overwrite, so they have to be zero; a
// caller who names the number of segments gets those.
bool prefill_short_built(const dsla_desc &d)
{
    return d.io_dtype == DSLA_F32 && d.segments == 0 && d.zero_init &&
           static_cast<int64_t>(d.H) * d.d_k * 16 * 4 < (int64_t{1} << 31);   // 32-bit offsets inside a tile
}

// Estimate (us): a launch, and the longer of the workgroup with the most keys and of all workgroups spread over the compute units,
// one to each.  Measured at d = 64, 4 heads of 64, 256, 512, 1000 tokens 6.3, 10.5, 16.8, 29.6, 32 heads of 64, 256, 512 6.5, 21.7, 50.9,
// 256 heads of 64, 256 42, 179; d = 128, 8 heads of 256, 512, 1000 18.2, 32.2, 82, 32 heads of 64, 256, 512 14.7, 38.8, 101; pre-activations
// 1.1 and 1.22 times that.
double prefill_short_cost(const dsla_desc &d, int64_t T)
{
    const bool small = d.d_k == 64;
    const double t = static_cast<double>(T), pre = d.gate_mode != DSLA_GATE_PREACT ? 1.0 : small ? 1.1 : 1.22;
    double groups = static_cast<double>(d.B) * d.H * (static_cast<double>((T + 15) / 16) + 2 * (d.d_k / 32)) / 256;
    if (T <= 64) groups = static_cast<double>(static_cast<int64_t>(groups + 0.999));   // (of about the same length: whole rounds)
    const double all = groups <= 1.0 ? 0.0 : groups * (small ? 4.4 + 0.0135 * t : 5.5 + 0.029 * t), longest = small ? 3.2 + 0.0225 * t : 4.5 + 0.049 * t;
    return 2.5 + pre * (all > longest ? all : longest);
}

hipError_t launch_prefill_short(const dsla_desc &d, const PrefillArgs &a, hipStream_t stream)
{
    const bool g16 = d.gate_dtype == DSLA_BF16;
    if (d.d_k == 128) return g16 ? launch<128, bf16_t>(a, d.B, stream) : launch<128, float>(a, d.B, stream);
    return g16 ? launch<64, bf16_t>(a, d.B, stream) : launch<64, float>(a, d.B, stream);
}

}  // namespace dsla
