// The projections in front of a DSLA layer as one MFMA GEMM (paper Section 5.3: "single linear layers for gating";
// appendix on training details: the q, k, v projections are the teacher's own, the history gate's weight starts near
// the identity, the recency gate's from a normal distribution, biases zero): from the layer input x [M][K]
// (M = batch * tokens, K = model width) and the stacked weights W [n_out * width][K] it writes n_out tensors
// [M][width] - q, k, v and the two gate pre-activations - each laid out [B][T][H][d] as the prefill reads them, so
// nothing is permuted or converted in between; with gate_mode = DSLA_GATE_PREACT the prefill applies the gate map.
//     out_j[m][c] = sum_k x[m][k] W[j * width + c][k] (+ bias[j * width + c])
// bf16 operands, fp32 accumulation, bf16 results.  Kernels (launch_project has the rule):
//
// project_tile_kernel<4> (K a multiple of 128): workgroup = 256 threads = 4 wavefronts on a 256 x 256 output tile, one
// wavefront per SIMD with a 128 x 128 quadrant = 8 x 8 MFMA tiles of 16 x 16 whose 256 accumulator registers live in
// the accumulation half of the register file.  Per 32 values of K a wavefront reads 8 + 8 fragments from LDS for 64
// MFMAs, which keeps the LDS out of the way.  K in stages of 32 through a ring of four LDS stages (4 x 32 KB),
// filled by buffer loads that write LDS directly (no staging registers, no LDS store instructions): a load has two
// stages to arrive.  Bound by power: the chip runs it at 1.8 GHz with the matrix pipes 73 % busy, and what an MFMA draws
// decides - registers only, 16 x 16 x 32 sustains 2.04 PFLOP/s and 32 x 32 x 16 1.77 (fewer accumulators are read and written
// per product).  M = 16384, K = 4096, N = 20480: 2.29 ms on 32 x 32 x 16, 2.09 on 16 x 16 x 32, 1.98 with the tile order
// below (1390 TFLOP/s; a plain library product of this shape 1.87 ms); with other inputs each time 2.34 ms before and 2.09 to 2.15 now;
// M = 4096 0.54, 0.49, 0.48 ms.
// A row of a stage is 64 bytes; its piece c sits at piece position c ^ 2 (row / 8 % 2).  A 16-byte LDS read takes lanes 0-3,
// 12-15, 20-27 at one time, then 4-11, 16-19, 28-31, and so on (32-63 alike): with this placement each of those
// sixteen finds its own four banks (no conflicts; with c ^ (row / 4 % 4), made for sixteen lanes in a row, every read took
// half as long again).  Tried and left out: a barrier every two stages (loads then have one and a half stages to arrive:
// 2.31 against 2.13 ms), tiles one after the other on a persistent grid with the next tile's stages loaded under
// the results' stores (2.17 against 2.08 ms: 512 registers do not hold it without spills).
//
// project_tile_kernel<2, 1>: the same on 128 x 128 tiles, two workgroups per compute unit, for outputs that do not fill the
// chip with large tiles.
//
// project_tile_kernel<1, 2>: 64 x 64 tiles and stages of 64 values of K, for outputs that do not fill it with those either.  A
// step of the 128 x 128 tiles takes 0.25 us however few there are (256 cycles of MFMAs behind a barrier and the LDS), so K = 4096
// took 33 us for 129 as for 1500 rows of 1536 columns; here a stage twice as long in K has a quarter of the MFMAs, and four
// times as many compute units share the work.  M = 300, K = 4096, N = 1536: 33.4 -> 17.8 us; M = 128, K = 2048, N = 5120 21.5 -> 10.7
// (row kernel before); M = 200, K = 1024, N = 3072 8.2 -> 5.1; M = 512, K = 4096, N = 1536 34.1 -> 18.8.  Tried: stages of 32 values in
// eight slots (the same within 5 %), of 128 in four (one workgroup per compute unit, 2 to 40 % slower), the 128 x 128 tiles with
// eight slots or stages of 64 (31 instead of 33 us), K split over the wavefronts with fragments straight from memory to
// registers (33 us for one 64 x 64 tile of K = 4096: 16 rows per load instruction run at 33 KB per us and compute unit).
//
// project_rows_kernel: up to 128 rows of x (the tokens of a decoding batch), where reading the weights is the work.
//
// project_kernel (more rows, K not a multiple of 128): 128 x 128 tile, 64 x 64 quadrants, K in steps of 32.
//
// Tile order of the tile kernels: see tile_of().
#include "dsla_internal.h"

#include <type_traits>

namespace dsla {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TM = 128, TN = 128, TK = 32;
constexpr int PITCH = TK + 8;   // elements per LDS row: 80 bytes, conflict-free for the 16-byte fragment reads

struct ProjectOuts {
    void *p[DSLA_MAX_PROJECTIONS];
};

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    f32x2 x = {a, b};
    bf16x2 y = __builtin_convertvector(x, bf16x2);
    return __builtin_bit_cast(uint32_t, y);
}

// 16 bytes per lane from a buffer (lane offset `voff`, uniform offset `soff`) into LDS at `lds` (uniform) + 16 * lane
__device__ __forceinline__ void buffer_load_lds16(__amdgpu_buffer_rsrc_t res, char *lds, uint32_t voff, int soff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(res, (__attribute__((address_space(3))) void *)(lds), 16, voff, soff, 0, 0);
}
template <int N>
__device__ __forceinline__ void wait_loads()   // at most N of this wavefront's loads are still in flight
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Tile order: the 8 XCDs each take a contiguous run of the linear tile order (workgroup ids go round-robin over the
// XCDs, each XCD has its own L2), and the linear order runs in groups of GM row tiles: inside a group the row tile
// runs fastest, then the column tile, so the tiles in flight at one time (a few dozen per XCD) share GM panels of x
// and a handful of panels of W instead of one panel of W and dozens of x.  M = 16384, K = 4096, N = 20480 with GM = 4, 6, 8,
// 16: 1.98, 1.99, 2.09, 2.24 ms.  Each group reads all of W, so a last group of one or two row tiles after a single full
// one is worth avoiding (group_rows()): M = 1060, K = 11008, N = 20480 in 4 + 1 and 5 row tiles 562 and 509 us.
// False: no tile for this workgroup.
__device__ __forceinline__ bool tile_of(int tiles_m, int tiles_n, int GM, long long per_xcd, int &tm, int &tn)
{
    const long long ntiles = static_cast<long long>(tiles_m) * tiles_n;
    const long long lin = static_cast<long long>(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (lin >= ntiles) return false;
    const long long per_group = static_cast<long long>(GM) * tiles_n;
    const int first_m = static_cast<int>(lin / per_group) * GM;
    const int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM;
    const int in_group = static_cast<int>(lin % per_group);
    tn = in_group / gsz;
    tm = first_m + in_group % gsz;
    return true;
}

// One 32 x 32 result tile, held transposed (tile rows = output columns): register r of lane (ln, g) is output row
// m_tile + ln, output column n_tile + 8 (r / 4) + 4 g + r % 4, so a lane stores 4 adjacent columns at a time.
__device__ __forceinline__ void store_tile(const f32x16 &acc, const ProjectOuts &outs, const float *__restrict__ bias,
                                           long long m, int n_tile, int g, int width, int N)
{
#pragma unroll
    for (int rb4 = 0; rb4 < 4; ++rb4) {
        const int col = n_tile + 8 * rb4 + 4 * g;   // 4 adjacent columns, inside one output tensor
        if (col >= N) continue;
        float c0 = acc[4 * rb4], c1 = acc[4 * rb4 + 1], c2 = acc[4 * rb4 + 2], c3 = acc[4 * rb4 + 3];
        if (bias) {
            c0 += bias[col];
            c1 += bias[col + 1];
            c2 += bias[col + 2];
            c3 += bias[col + 3];
        }
        bf16_t *dst = static_cast<bf16_t *>(outs.p[col / width]) + static_cast<size_t>(m) * width + col % width;
        *reinterpret_cast<u32x2 *>(dst) = u32x2{pack2(c0, c1), pack2(c2, c3)};
    }
}

// ---------------------------------------------------------------------------------------------------------------
// 256 x 256 and 128 x 128 tiles, loads straight into LDS
// ---------------------------------------------------------------------------------------------------------------
constexpr int BK = 32;                            // values of K per stage
constexpr int ROWB = BK * 2;                     // bytes per LDS row: 64

// Q: 32 x 32 tiles along each side of a wavefront's quadrant (4: 256 x 256 per workgroup, 2: 128 x 128, 1: 64 x 64); KS: blocks
// of 32 values of K per stage
template <int Q, int KS>
__global__ __launch_bounds__(256, Q == 4 ? 1 : 2) void project_tile_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w,
                                                                 const float *__restrict__ bias, ProjectOuts outs, long long M,
                                                                 int K, int N, int width, int tiles_m, int tiles_n, int group,
                                                                 long long per_xcd)
{
    constexpr int BM = 64 * Q, BN = BM, QS = 32 * Q;   // workgroup tile, quadrant
    constexpr int OPB = BM * ROWB;                      // bytes per operand tile and block of 32 values of K
    constexpr int STAGEB = 2 * OPB * KS;                // KS times: A tile, then B tile
    // four stages as four objects: the compiler's wait-count insertion then knows that a load into one stage does not
    // touch what is read from another
    __shared__ __attribute__((aligned(1024))) char st0[STAGEB];
    __shared__ __attribute__((aligned(1024))) char st1[STAGEB];
    __shared__ __attribute__((aligned(1024))) char st2[STAGEB];
    __shared__ __attribute__((aligned(1024))) char st3[STAGEB];
    int tm, tn;
    if (Q > 1 || group > 0) {
        if (!tile_of(tiles_m, tiles_n, group, per_xcd, tm, tn)) return;
    } else if (!tile_of(tiles_n, tiles_m, -group, per_xcd, tn, tm)) {
        return;
    }
    const long long m0 = static_cast<long long>(tm) * BM;
    const int n0 = tn * BN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;   // this wavefront's quadrant
    const uint32_t uwave = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(wave));

    // Buffer loads with LDS as destination: one instruction of a wavefront fills 1 KB = 16 rows of 64 bytes of a
    // tile; instruction n = wave + 4 i (i < Q) fills rows 16 n .. 16 n + 15.  A lane fills LDS slot (row lane / 4, piece
    // position lane % 4) and fetches the piece that belongs there (piece c of row R sits at c ^ 2 (R / 8 % 2)).  The
    // descriptor of an operand starts at the tile's first row and ends with the last row that exists: rows past the
    // end of x or W arrive as zeros.
    const long long rows_a = M - m0 < BM ? M - m0 : BM, rows_b = N - n0 < BN ? N - n0 : BN;
    const __amdgpu_buffer_rsrc_t res_a = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(x + static_cast<size_t>(m0) * K), 0, static_cast<int>(rows_a * K * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t res_b = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(w + static_cast<size_t>(n0) * K), 0, static_cast<int>(rows_b * K * 2), 0x00020000);
    uint32_t voff[Q];   // byte offset of this lane's piece from the first row of the tile (the range check is on it)
#pragma unroll
    for (int i = 0; i < Q; ++i)
        voff[i] = (16 * (uwave + 4 * i) + (static_cast<uint32_t>(lane) >> 2)) * static_cast<uint32_t>(K) * 2u +
                  16 * ((lane & 3u) ^ (((static_cast<uint32_t>(lane) >> 5) & 1u) << 1));
    const int nk = K / (BK * KS);
    auto fetch = [&](char *st, int ks) {   // K-step ks (past the end: the last one again, never used) into a stage
        const int kbyte = (ks < nk ? ks : nk - 1) * (BK * KS * 2);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const uint32_t n = uwave + 4 * i;
                buffer_load_lds16(res_a, st + kk * 2 * OPB + n * 1024, voff[i], kbyte + kk * BK * 2);
                buffer_load_lds16(res_b, st + kk * 2 * OPB + OPB + n * 1024, voff[i], kbyte + kk * BK * 2);
            }
    };

    // fragment reads: row (quadrant + 16 i + r) of a tile, values 8 g .. 8 g + 7 of the stage: piece g
    constexpr int NF = 2 * Q;   // 16 x 16 tiles along each side of the quadrant
    const uint32_t fo = (g ^ ((r >> 3) << 1)) << 4;
    const uint32_t fa_row = static_cast<uint32_t>((QS * wm + r) * ROWB) + fo;
    const uint32_t fb_row = static_cast<uint32_t>(OPB + (QS * wn + r) * ROWB) + fo;
    struct Frags {
        bf16x8 a[KS][NF], b[KS][NF];
    };
    auto read_frags = [&](Frags &f, const char *st) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                f.a[kk][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(st + kk * 2 * OPB + fa_row + i * 16 * ROWB));
                f.b[kk][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(st + kk * 2 * OPB + fb_row + i * 16 * ROWB));
            }
    };

    f32x4 acc[NF][NF];
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // One K-step.  On entry its fragments are in registers (or on their way) and stage `nxt` holds
    // what this wavefront loaded of the next step but one barrier short of being complete for everybody: the barrier
    // at the start certifies `nxt` (every wavefront has waited for its own loads of it: all but the 2 Q youngest, which
    // belong to the stage after) and frees `old` (everybody has multiplied the step before, so nobody reads it any more),
    // which then takes K-step ks + 3.  So a load has two steps to arrive, and the fragments of `nxt` are read under the
    // MFMAs of the current step.
    auto step = [&](const Frags &cur, Frags &nf, const char *nxt, char *old, int ks) {
        wait_loads<2 * Q * KS>();
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        fetch(old, ks + 3);
        read_frags(nf, nxt);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int i = 0; i < NF; ++i)
#pragma unroll
                for (int j = 0; j < NF; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur.b[kk][j], cur.a[kk][i], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < 2 * NF * KS; ++t) {
            __builtin_amdgcn_sched_group_barrier(0x008, NF / 2 - NF / 4, 0);        // MFMAs
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                      // 1 LDS read
            if (NF >= 4) __builtin_amdgcn_sched_group_barrier(0x008, NF / 4, 0);
            if (t % 2 == 0) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);      // 1 load into LDS
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // nk is a multiple of 4 (K is a multiple of 128 KS): the loop body has no branch, so the accumulators stay where they are
    fetch(st0, 0);
    fetch(st1, 1);
    fetch(st2, 2);
    wait_loads<4 * Q * KS>();
    asm volatile("s_barrier" ::: "memory");   // stage 0 is complete
    Frags f0, f1;
    read_frags(f0, st0);
    __builtin_amdgcn_sched_barrier(0);
    for (int ks = 0; ks < nk; ks += 4) {
        step(f0, f1, st1, st3, ks);
        step(f1, f0, st2, st0, ks + 1);
        step(f0, f1, st3, st1, ks + 2);
        step(f1, f0, st0, st2, ks + 3);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // nothing in flight; everybody is done reading

    // Results: each wavefront turns its quadrant round in LDS - its own stage object, 128 rows of 256 bytes, the 16-byte
    // piece c of row r at position c ^ (r % 16) - so that it leaves as whole rows: a lane holds 4 adjacent columns of a
    // row per register group and writes them as 8 bytes; then 16 lanes read one row as 16 bytes each and store 256
    // contiguous bytes.
    constexpr int PPR = QS / 8;   // 16-byte pieces per quadrant row
    char *epi = wave == 0 ? st0 : (wave == 1 ? st1 : (wave == 2 ? st2 : st3));
    const int nq = n0 + QS * wn;   // first column of the quadrant: inside one output tensor (width is a multiple of 128)
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int cq = 16 * j + 4 * g;   // column inside the quadrant
            f32x4 c = acc[i][j];
            if (bias && nq + cq < N) {
                const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias + nq + cq);
#pragma unroll
                for (int e = 0; e < 4; ++e) c[e] += bv[e];
            }
            const int row = 16 * i + r, piece = cq >> 3;
            *reinterpret_cast<u32x2 *>(epi + row * (2 * QS) + ((piece ^ (row & (PPR - 1))) << 4) + (cq & 4) * 2) = u32x2{pack2(c[0], c[1]), pack2(c[2], c[3])};
        }
    if (nq < N) {
        bf16_t *out = static_cast<bf16_t *>(outs.p[nq / width]) + nq % width;
        const int rsub = lane / PPR, piece = lane % PPR;   // PPR lanes per row
#pragma unroll 4
        for (int it = 0; it < QS * PPR / 64; ++it) {
            const int row = 64 / PPR * it + rsub;
            const long long m = m0 + QS * wm + row;
            const u32x4 vrow = *reinterpret_cast<const u32x4 *>(epi + row * (2 * QS) + ((piece ^ (row & (PPR - 1))) << 4));
            if (m < M)   // streaming store: a tile of results is not read again by this kernel
                __builtin_nontemporal_store(vrow, reinterpret_cast<u32x4 *>(out + static_cast<size_t>(m) * width + piece * 8));
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// 128 x 128 tiles
// ---------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void project_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w,
                                                      const float *__restrict__ bias, ProjectOuts outs, long long M, int K,
                                                      int width, int tiles_m, int tiles_n, int group)
{
    __shared__ __attribute__((aligned(16))) bf16_t sA[2][TM * PITCH];
    __shared__ __attribute__((aligned(16))) bf16_t sB[2][TN * PITCH];

    int tm, tn;
    if (!tile_of(tiles_m, tiles_n, group, (static_cast<long long>(tiles_m) * tiles_n + 7) / 8, tm, tn)) return;
    const long long m0 = static_cast<long long>(tm) * TM;
    const int n0 = tn * TN;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ln = lane & 31, g = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;   // this wavefront's 64 x 64 quadrant

    // staging: 512 16-byte pieces per operand tile and K-step, two per thread: piece -> (row, 8 k-values)
    u32x4 ra[2], rb[2];
    auto load_tiles = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int piece = tid + 256 * i, row = piece >> 2, c = piece & 3;
            const long long m = m0 + row;
            ra[i] = u32x4{0, 0, 0, 0};
            if (m < M) ra[i] = *reinterpret_cast<const u32x4 *>(x + static_cast<size_t>(m) * K + k0 + 8 * c);
            rb[i] = *reinterpret_cast<const u32x4 *>(w + static_cast<size_t>(n0 + row) * K + k0 + 8 * c);
        }
    };
    auto store_tiles = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int piece = tid + 256 * i, row = piece >> 2, c = piece & 3;
            *reinterpret_cast<u32x4 *>(&sA[buf][row * PITCH + 8 * c]) = ra[i];
            *reinterpret_cast<u32x4 *>(&sB[buf][row * PITCH + 8 * c]) = rb[i];
        }
    };

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    const int nk = K / TK;
    load_tiles(0);
    store_tiles(0);
    for (int ks = 0; ks < nk; ++ks) {
        __syncthreads();   // K-step ks is in buffer ks & 1; every wavefront is done with step ks - 1
        if (ks + 1 < nk) load_tiles((ks + 1) * TK);
        const bf16_t *a = sA[ks & 1], *b = sB[ks & 1];
        // acc[i][j] holds C^T tiles: result tile rows = output columns (from W), tile columns = output rows (from x),
        // so that a lane ends up with 4 adjacent output columns of one output row: 8-byte stores
#pragma unroll
        for (int kb = 0; kb < TK / 16; ++kb) {
            bf16x8 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                fa[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(&a[(64 * wm + 32 * i + ln) * PITCH + 16 * kb + 8 * g]));
                fb[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(&b[(64 * wn + 32 * i + ln) * PITCH + 16 * kb + 8 * g]));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
        }
        if (ks + 1 < nk) store_tiles((ks + 1) & 1);
    }

#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const long long m = m0 + 64 * wm + 32 * i + ln;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) store_tile(acc[i][j], outs, bias, m, n0 + 64 * wn + 32 * j, g, width, tiles_n * TN);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Few rows: the weights are the traffic
// ---------------------------------------------------------------------------------------------------------------
// Bound by HBM: 2 N K bytes of weights.  Workgroup = 4 wavefronts on 16 MT rows of x (all of them: at most 128) and 16 NT
// columns (row_column_tiles() has the rule).  Stages of 64 KS values of K - KS lines of 128 bytes
// of each of the 16 (NT + MT) rows; whole lines, because a request costs the L2 the same whatever its size - go through
// a ring of LDS slots filled by loads that write LDS directly, so three stages are in flight whatever the registers
// hold.  The fragments of the next stage are read while the MFMAs of the current one run (without that a stage costs
// its LDS latency on top: M = 64 41.5 us instead of 34.5), and short stages are merged (KS) because the barrier of a
// stage costs about 0.2 us (M = 20, N = 3072, K = 4096: KS = 1 18.2, 2 12.9, 4 11.0 us).  One row tile and five column tiles keep
// stages of one line: with 48 KB three workgroups share a compute unit, with 96 KB one (M = 8, N = 28672, K = 512 8.4 against
// 10.6 us, K = 4096 48.5 against 50.5; N = 20480, which is one round either way, 6.3 against 6.7 and 31.2 against 31.8).
// K = 4096, N = 20480 (170 MB): M = 1 32 us = 5.3 TB/s, M = 64 34.5 us = 5.0 TB/s, M = 128 48 us; the 128 x 128 tiles take
// 56, 56 and 59 us, the 256 x 256 ones 80, 83 and 94.
template <int MT, int NT>
struct Rows {
    static constexpr int KS = MT + NT <= 3 ? 4 : (MT + NT > 12 || (MT == 1 && NT == 5) ? 1 : 2);   // lines of 64 values per row and stage
    static constexpr int LB = 2 * (NT + MT), L = LB * KS;                  // load instructions per stage: 8 rows of 128 bytes each
    static constexpr uint32_t BLOCK = LB * 1024, STAGE = L * 1024;
    static constexpr int DEPTH_MAX = 150 * 1024 / static_cast<int>(STAGE);
    static constexpr int DEPTH = DEPTH_MAX > 4 ? 4 : DEPTH_MAX;             // (six and eight slots: no difference)
    static constexpr int WM = MT < 4 ? MT : 4, WN = 4 / WM;      // wavefronts along the rows of x / along the columns
    static constexpr int TM_ = MT / WM, TN_ = (NT + WN - 1) / WN;   // tiles of a wavefront
};
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane from `base` (uniform) + `voff` (per lane) into LDS at `lds` (uniform) + 16 * lane; the compiler does
// not know these loads: whoever reads the bytes waits with wait_loads() first.
__device__ __forceinline__ void load_to_lds16(uint32_t lds, uint32_t voff, const char *base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "m0", "memory");
}
#pragma clang diagnostic pop

template <int MT, int NT>
__global__ __launch_bounds__(256) void project_rows_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ w,
                                                           const float *__restrict__ bias, ProjectOuts outs, int M, int K,
                                                           int N, int width)
{
    using R = Rows<MT, NT>;
    constexpr int DEPTH = R::DEPTH;
    __shared__ __attribute__((aligned(1024))) char ring[DEPTH * R::STAGE];
    const int n0 = blockIdx.x * 16 * NT;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const uint32_t ring_lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char *)ring));

    // ---- loading: instruction i of a stage fills rows 8 i .. 8 i + 7 (the 16 NT weight rows, then the rows of x), lane
    // l position l % 8 of row l / 8; piece c of a row sits at position c ^ ((row / 2) % 8), which spreads the 16 rows
    // that 16 lanes read at one piece over all banks.  Rows past the end re-read the last one (their results are not
    // stored).  Wavefront w issues instructions w, w + 4, ... ----
    constexpr int CMAX = (R::L + 3) / 4;
    const int ns = (K + 64 * R::KS - 1) / (64 * R::KS);
    const int last_units = K / 32 - (ns - 1) * 2 * R::KS;   // blocks of 32 values in the last stage; the others re-read its first
    const char *src[CMAX];
    uint32_t voff[CMAX], unit[CMAX];   // unit: which block of 32 values of the stage the lane's piece belongs to
#pragma unroll
    for (int c = 0; c < CMAX; ++c) {
        const int n = wave + 4 * c, i = n % R::LB;
        const uint32_t srow = 8 * i + (static_cast<uint32_t>(lane) >> 3), piece = (lane & 7u) ^ ((srow >> 1) & 7u);
        int row;
        if (i < 2 * NT) {
            row = static_cast<int>(srow);
            row = n0 + row < N ? row : N - 1 - n0;
        } else {
            row = static_cast<int>(srow) - 16 * NT;
            row = row < M ? row : M - 1;
        }
        voff[c] = static_cast<uint32_t>(row) * static_cast<uint32_t>(K) * 2u + 128 * (n / R::LB) + 16 * piece;
        unit[c] = 2 * (n / R::LB) + (piece >> 2);
        src[c] = reinterpret_cast<const char *>(i < 2 * NT ? w + static_cast<size_t>(n0) * K : x);
    }
    // Workgroups start their walk at different stages, so that the lines they ask for at one time spread over the memory
    // channels (rows are a large power of two apart; M = 16: 35.0 us when all start at stage 0, 29.8 us).
    const int rot = (3 * (blockIdx.x / 8)) % ns;
    auto issue = [&](int i, int at) {   // stage i of the walk into ring slot `at`
        int s = i + rot;
        s = s < ns ? s : s - ns;
        const uint32_t units = s == ns - 1 ? last_units : 2 * R::KS;
#pragma unroll
        for (int c = 0; c < CMAX; ++c) {
            const int n = wave + 4 * c;
            if (n < R::L)
                load_to_lds16(ring_lds + at * R::STAGE + n * 1024, unit[c] < units ? voff[c] : voff[c] - 64 * unit[c],
                              src[c] + static_cast<size_t>(s) * (128 * R::KS));
        }
    };

    // ---- fragments: lane (r, g) holds row r, values 8 g .. of a block of 32 ----
    const int r = lane & 15, g = lane >> 4, wm = wave % R::WM, wn = wave / R::WM;
    const uint32_t fpos[2] = {((0u + g) ^ ((r >> 1) & 7u)) << 4, ((4u + g) ^ ((r >> 1) & 7u)) << 4};
    f32x4 acc[R::TM_][R::TN_];
#pragma unroll
    for (int i = 0; i < R::TM_; ++i)
#pragma unroll
        for (int j = 0; j < R::TN_; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Frags {
        bf16x8 x[2 * R::KS][R::TM_], w[2 * R::KS][R::TN_];
    };
    auto read = [&](Frags &f, int at) {
#pragma unroll
        for (int kk = 0; kk < 2 * R::KS; ++kk) {
            const char *st = ring + at * R::STAGE + (kk >> 1) * R::BLOCK + r * 128;
#pragma unroll
            for (int a = 0; a < R::TM_; ++a)
                f.x[kk][a] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(st + (NT + wm + R::WM * a) * 2048 + fpos[kk & 1]));
#pragma unroll
            for (int b = 0; b < R::TN_; ++b) {
                const int t = wn + R::WN * b;   // (a wavefront with one tile less repeats the last one and drops it)
                f.w[kk][b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(st + (t < NT ? t : NT - 1) * 2048 + fpos[kk & 1]));
            }
        }
    };
    auto mma = [&](const Frags &f, int kk) {   // result transposed: lane (r, g) holds row r of x, columns 4 g .. 4 g + 3
#pragma unroll
        for (int b = 0; b < R::TN_; ++b)
#pragma unroll
            for (int a = 0; a < R::TM_; ++a)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.w[kk][b], f.x[kk][a], acc[a][b], 0, 0, 0);
    };

    constexpr int REM = R::L % 4, CLO = R::L / 4, CHI = REM ? CLO + 1 : CLO;
    auto arrive = [&](bool full) {   // all but the DEPTH - 2 youngest stages of every wavefront's loads are in LDS
        if (!full) wait_loads<0>();
        else if (REM && wave < REM) wait_loads<CHI * (DEPTH - 2)>();
        else wait_loads<CLO * (DEPTH - 2)>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
#pragma unroll
    for (int i = 0; i < DEPTH - 1; ++i)
        if (i < ns) issue(i, i);
    arrive(DEPTH - 2 < ns);   // stage 0 has landed
    Frags f0, f1;
    read(f0, 0);
    if (DEPTH - 1 < ns) issue(DEPTH - 1, DEPTH - 1);
    int at = 0;   // slot of stage i
    auto step = [&](const Frags &cur, Frags &nxt, int i) {
        const int at_n = at + 1 == DEPTH ? 0 : at + 1;
        if (i + 1 < ns) {
            // stage i + 1 has landed; everybody holds the fragments of stage i, whose slot takes stage i + DEPTH
            arrive(i + DEPTH - 1 < ns);
            if (i + DEPTH < ns) issue(i + DEPTH, at);
            read(nxt, at_n);
        }
        int s = i + rot;
        s = s < ns ? s : s - ns;
        const int units = s == ns - 1 ? last_units : 2 * R::KS;
#pragma unroll
        for (int kk = 0; kk < 2 * R::KS; ++kk)
            if (kk == 0 || kk < units) mma(cur, kk);
        at = at_n;
    };
    for (int i = 0; i < ns; i += 2) {
        step(f0, f1, i);
        if (i + 1 < ns) step(f1, f0, i + 1);
    }
#pragma unroll
    for (int a = 0; a < R::TM_; ++a) {
        const int m = 16 * (wm + R::WM * a) + r;
        if (m >= M) continue;
#pragma unroll
        for (int b = 0; b < R::TN_; ++b) {
            const int t = wn + R::WN * b, col = n0 + 16 * t + 4 * g;
            if (t >= NT || col >= N) continue;
            f32x4 s = acc[a][b];
            if (bias) {
                const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias + col);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] += bv[e];
            }
            bf16_t *dst = static_cast<bf16_t *>(outs.p[col / width]) + static_cast<size_t>(m) * width + col % width;
            *reinterpret_cast<u32x2 *>(dst) = u32x2{pack2(s[0], s[1]), pack2(s[2], s[3])};
        }
    }
}

}  // namespace

namespace {
// Row tiles per group of the tile order: four, or all of them up to `whole`.
int group_rows(int tiles_m, int whole) { return tiles_m <= whole ? tiles_m : 4; }
// Of the 64 x 64 tiles.  A tile that does not find its neighbours (the same columns of W) in its XCD's L2 waits for memory in every
// step, and with one tile to a compute unit the slowest is the call.  Two row tiles: runs of whole pairs (M = 96, K = 7936,
// N = 2816 37.4 us with pairs split between two XCDs, 35.4 in the row kernel, 30.5 so).  More tiles than units, up to 15 row tiles: all of
// them are one group, in runs of whole columns (M = 371, K = 1536, N = 3456 in 4 + 2 and 6 row tiles 14.3 and 10.7 us, 128 x 128
// tiles 10.9; M = 960, K = 2048, N = 1152 in 4 + 4 + 4 + 3 and 15 16.7 and 13.5, 12.9); up to 15 column tiles: the same the other way
// round, runs of whole rows, which share those of x (a negative group; M = 1959, K = 2048, N = 640 17.5 and 13.0, 13.7).  800 random products
// of 257 to 400 tiles: slower than 128 x 128 tiles by more than 3 % in about 1 of 100 (16 and more tiles both ways, or K = 8192), in
// groups of four in 16 of 100.  Not for K >= 4096, where the tiles of a column drift apart (K = 8192 2.5 % slower on average), nor for
// up to 256 tiles of three and more row tiles, where a whole column may be one tile too many for an XCD's 32 units (up to 26 %).
void tile_order(int tiles_m, int tiles_n, int K, int &group, int &unit)
{
    const bool many = K < 4096 && static_cast<long long>(tiles_m) * tiles_n > 256;
    group = group_rows(tiles_m, 5);
    unit = tiles_m == 2 ? group : 1;
    if (many && tiles_m <= 15) {
        group = unit = tiles_m;
    } else if (many && tiles_n <= 15) {
        group = -tiles_n;
        unit = tiles_n;
    }
}

template <int MT, int NT>
void launch_rows(ProfileScope &ps, int M, int K, int N, int width, const void *x, const void *w, const float *bias,
                 const ProjectOuts &po, hipStream_t stream)
{
    const unsigned grid = static_cast<unsigned>((N + 16 * NT - 1) / (16 * NT));   // one workgroup has all rows: M <= 16 MT
    DSLA_LAUNCH(ps, (project_rows_kernel<MT, NT>), dim3(grid), dim3(256), 0, stream, static_cast<const bf16_t *>(x),
                static_cast<const bf16_t *>(w), bias, po, M, K, N, width);
}
// Column tiles per workgroup of the row kernel: the most that still leave 256 workgroups, one for every compute unit, of the
// numbers that are built: 1, 2, 3 and 5 (from N = 4096 times that number).  Between 12288 and 20479 columns, where four would be
// the number, three make up to 426 workgroups: M = 64, K = 4096, N = 16384 43 us against 34 at N = 20480.
int row_column_tiles(int N)
{
    const int nt = N / (16 * 256);
    return nt >= 5 ? 5 : (nt >= 3 ? 3 : (nt == 2 ? 2 : 1));
}
int row_workgroups(int N)
{
    const int columns = 16 * row_column_tiles(N);
    return (N + columns - 1) / columns;
}
template <int MT>
void launch_rows_n(ProfileScope &ps, int M, int K, int N, int width, const void *x, const void *w, const float *bias,
                   const ProjectOuts &po, hipStream_t stream)
{
    const int nt = row_column_tiles(N);
    if (nt == 5) launch_rows<MT, 5>(ps, M, K, N, width, x, w, bias, po, stream);
    else if (nt == 3) launch_rows<MT, 3>(ps, M, K, N, width, x, w, bias, po, stream);
    else if (nt == 2) launch_rows<MT, 2>(ps, M, K, N, width, x, w, bias, po, stream);
    else launch_rows<MT, 1>(ps, M, K, N, width, x, w, bias, po, stream);
}
template <int Q, int KS>
void launch_tiles(ProfileScope &ps, int64_t M, int K, int N, int width, const void *x, const void *w, const float *bias,
                  const ProjectOuts &po, hipStream_t stream)
{
    constexpr int B = 64 * Q;
    const int tiles_m = static_cast<int>((M + B - 1) / B), tiles_n = (N + B - 1) / B;
    const long long ntiles = static_cast<long long>(tiles_m) * tiles_n;
    int group = group_rows(tiles_m, 5), unit = 1;
    if (Q == 1) tile_order(tiles_m, tiles_n, K, group, unit);
    const long long per_xcd = ((ntiles + 7) / 8 + unit - 1) / unit * unit;
    const unsigned grid = static_cast<unsigned>(8 * per_xcd);
    DSLA_LAUNCH(ps, (project_tile_kernel<Q, KS>), dim3(grid), dim3(256), 0, stream, static_cast<const bf16_t *>(x),
                static_cast<const bf16_t *>(w), bias, po, static_cast<long long>(M), K, N, width, tiles_m, tiles_n,
                group, per_xcd);
}
}  // namespace

hipError_t launch_project(int64_t M, int K, int n_out, int width, const void *x, const void *w, const float *bias,
                          void *const *outs, hipStream_t stream)
{
    ProjectOuts po;
    for (int j = 0; j < DSLA_MAX_PROJECTIONS; ++j) po.p[j] = j < n_out ? outs[j] : nullptr;
    const int N = n_out * width;
    ProfileScope ps(DSLA_KERNEL_PROJECT, stream);
    // Few rows: the weights are the traffic.  Not where the row kernel's workgroups need a second, nearly empty round over the
    // compute units and the others pass the weights in one: with 65 .. 128 rows N = 24576, K = 4096 86 / 59 us (row kernel /
    // 128 x 128 tiles), N = 16384, K = 2048 34 / 30, but N = 20480 47 / 58 and 27 / 31 (K = 1024: 17 / 13, where the tile
    // kernel's stages are few); where K is no multiple of 128, N = 28672, K = 160 13 / 10, K = 480 20 / 18, K = 1056 31 / 32.
    // Up to 64 rows a second round is the lesser evil, except for the shortest K: N = 28672, K = 160 10.6 / 9.3, K = 480 16 / 18.
    // (Past 32768 columns the others' tiles go twice over the chip as well: N = 35840, K = 4096, 97 rows 87 / 99.)
    const bool second_round = N > 12288 && N <= 32768 && row_workgroups(N) > 256;
    // 64 x 64 tiles while they find compute units of their own, against the 128 x 128 ones also where a few units get two.  Row
    // kernel or 128 x 128 / 64 x 64 tiles (us): 160 tiles 21.5 / 10.7 and 33.2 / 17.2, 240 10.5 / 6.4, 264 34.0 / 29.2, 320 34.2 / 32.0
    // and 18.3 / 13.6, 384 11.3 / 10.7, 400 18.5 / 16.2, but 528 11.5 / 14.7 and 640 34.9 / 46.7; up to 128 rows 384 tiles 16.9 / 14.3
    // and 17.4 / 18.5, and at K = 512 288 tiles 6.0 / 6.7, 320 6.1 / 5.6, 360 6.2 / 6.6.  Up to 64 rows the row kernel reads the weights as fast or faster.
    const int64_t tiles64 = (M + 63) / 64 * (N / 64);
    if (M > 64 && K % (8 * BK) == 0 && tiles64 <= (M <= 128 ? 256 : (K >= 1024 ? 400 : 256))) {
        launch_tiles<1, 2>(ps, M, K, N, width, x, w, bias, po, stream);
    } else if (M <= 16 || (M <= 64 && (N <= 20480 || K >= 256)) ||
        (M > 64 && M <= 128 && (K % (4 * BK) == 0 ? K >= 2048 && !second_round : K >= 1024 || !second_round))) {
        const int m = static_cast<int>(M);
        if (M <= 16) launch_rows_n<1>(ps, m, K, N, width, x, w, bias, po, stream);
        else if (M <= 32) launch_rows_n<2>(ps, m, K, N, width, x, w, bias, po, stream);
        else if (M <= 64) launch_rows_n<4>(ps, m, K, N, width, x, w, bias, po, stream);
        else launch_rows_n<8>(ps, m, K, N, width, x, w, bias, po, stream);
    } else if (K % (4 * BK) == 0) {   // the loop of project_tile_kernel goes four stages at a time
        // Small tiles while the chip has compute units for them: the rounds over the 256 compute units decide.  A large tile does
        // four times the work of a small one in 2.2 times its time where K is long; where it is short the epilogue weighs
        // more, 2.8 times at K = 512.  Small / large (us): K = 4096: M = 384, N = 20480 95 / 102; M = 1300, N = 3072 59 / 77;
        // M = 640, N = 20480 154 / 114; M = 1480, N = 12288 189 / 174; K = 11008: M = 520, N = 28672 521 / 459; K = 512:
        // M = 2600, N = 12288 45 / 56, M = 384, N = 28672 26 / 21.
        const int64_t rounds128 = ((M + 127) / 128 * (N / 128) + 255) / 256;
        const int64_t rounds256 = ((M + 255) / 256 * ((N + 255) / 256) + 255) / 256;
        if (10 * rounds128 * K <= (22 * static_cast<int64_t>(K) + 3200) * rounds256) launch_tiles<2, 1>(ps, M, K, N, width, x, w, bias, po, stream);
        else launch_tiles<4, 1>(ps, M, K, N, width, x, w, bias, po, stream);
    } else {
        const int tiles_m = static_cast<int>((M + TM - 1) / TM), tiles_n = N / TN;
        const long long ntiles = static_cast<long long>(tiles_m) * tiles_n;
        const unsigned grid = static_cast<unsigned>((ntiles + 7) / 8 * 8);
        DSLA_LAUNCH(ps, project_kernel, dim3(grid), dim3(256), 0, stream, static_cast<const bf16_t *>(x),
                           static_cast<const bf16_t *>(w), bias, po, static_cast<long long>(M), K, width, tiles_m, tiles_n,
                           group_rows(tiles_m, 6));
    }
    return hipGetLastError();
}

}  // namespace dsla
