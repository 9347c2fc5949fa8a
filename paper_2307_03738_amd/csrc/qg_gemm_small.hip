// qg_gemm_small: Y = X What^T for a few prompt tokens (M <= 128) on the matrix cores.
//
// The paper treats only the vector input; this is the same What = s (q - z) (Section 2,
// eq. (1)) applied to M activation rows at once.  X and the dequantized weights are rounded
// to bf16, products are accumulated in fp32 by v_mfma_f32_32x32x16_bf16.
//
// Mapping (4-bit codes, groups of 32, 64, 128 or a multiple of 128).  A wavefront owns one
// tile of 64 outputs -- the same device layout the GEMV reads, lane l holding 32 consecutive
// k of output 64*tile + l in one 128-bit vector -- and all M rows.  The matrix instruction
// wants, for a block of 32 outputs, lanes l and l+32 to hold the SAME output with two
// different k-octets; the layout has them hold two different outputs with the same k.  One
// v_permlane32_swap of the raw code words (w0 with w2, w1 with w3) turns one into the other
// for both 32-output blocks at once, so weights go from HBM to the MFMA operand through
// registers only: mask, convert, one FMA with the group's (s, -z s), pack to bf16.  Every
// weight is dequantized exactly once.
//
// A wavefront holds at most 64 activation rows (64 accumulator registers); more rows run as
// two row blocks on the grid's z axis.  A workgroup is four wavefronts laid out as TN tiles x
// KW k-slices (TN * KW = 4): four neighbouring tiles over the same k (KW = 1) when the launch
// has enough workgroups anyway, otherwise two or four consecutive k-steps of fewer tiles
// (KW = 2, 4), whose accumulators are added through LDS at the end -- more wavefronts for
// small problems without more partial results.  The activation rows are converted to bf16
// on their way into LDS, KW * 128 k at a time, double-buffered, shared by the workgroup; the
// loads of the next chunk are issued a quarter at a time between the units of the running
// step, because the path from L2 into a compute unit is what the activations load most.
// Codes, scales and zero-points of the next step are in flight while the current one is
// computed.  K may also be cut into `splits` ranges handled by different workgroups; their
// fp32 partial results are added by a second small kernel in a fixed order.
//
// The other widths, 4-bit groups of 16 and the larger 4-bit products take the kernel on raw codes
// (qg_gemm_codes.h), 3-bit groups of 32 the one on int8 digits (qg_gemm_rows_i8.hip); what none of them takes, and
// few rows of small matrices, runs the fp32 GEMV kernel once per activation row, up to 16 rows per launch.
#include <cmath>
#include <mutex>
#include <type_traits>

#include "qg_common.h"
#include "qg_gemm_codes.h"
#include "qg_mma.h"

size_t qg_gemm_workspace_bytes(const QgLayout &L, int M);
int qg_gemm_rows16(const void *packed, int64_t N, int64_t K, int bits, int group, const float *X,
                   int M, float *Y, void *workspace, void *stream, bool dry);   // qg_gemv.hip
bool qg_rows_i8_takes(const QgLayout &L);                 // qg_gemm_rows_i8.hip
size_t qg_rows_i8_bytes(const QgLayout &L, int M);
int qg_rows_i8_splits(const QgLayout &L, int M);
double qg_rows_i8_us(const QgLayout &L, int M);
int qg_rows_i8(const void *packed, const QgLayout &L, const float *X, int M, float *Y, void *workspace, hipStream_t st, float **partial);
int qg_gemv_rows(const void *packed, int64_t N, int64_t K, int bits, int group, const float *X, int M, float *Y,
                 void *stream, bool dry);
int qg_gemv_grouped_rows(const qg_gemv_desc *descs, int count, void *workspace, size_t workspace_bytes, void *stream);
int qg_gemv_grouped_check(const qg_gemv_desc *descs, int count, void *workspace, size_t workspace_bytes);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int KC = 128;            // k per step of the 4-bit layout
constexpr int MAX_SPLITS = 8;      // partial results per element of Y

struct GemmArgs {
    const uint4 *codes;
    const float *scales;
    const uint32_t *zeros;
    const float *X;            // activations [M][K] fp32
    float *out;                // Y, or partial results [split][M][N]
    int M, N, K, tiles, steps, ngroups, zwords;
    int group_shift;           // log2(G) for G <= 128
    int steps_per_group;       // G / 128 for G > 128, else 1
    int steps_per_split;       // a multiple of KW and of steps_per_group
};

__device__ inline uint32_t opaque(uint32_t v)
{
    asm("" : "+v"(v));
    return v;
}

union Operand {
    bf16x8 v;
    bf16x2 p[4];
};

// Eight 4-bit codes of one word -> eight bf16 values s*(q - z), in code order.  The odd codes
// are taken with one mask, sixteen times too large, and multiplied by s / 16 (exact).
__device__ inline bf16x8 dequant_word(uint32_t w, float s, float nzs)
{
    const uint32_t lo = opaque(w & 0x0f0f0f0fu);          // codes 0, 2, 4, 6
    const uint32_t hi = opaque(w & 0xf0f0f0f0u);          // codes 1, 3, 5, 7, times 16
    const float sh = s * 0.0625f;
    Operand o;
    floatx2 t;
    t[0] = fmaf((float)(lo & 0xffu), s, nzs);          t[1] = fmaf((float)(hi & 0xffu), sh, nzs);
    o.p[0] = __builtin_convertvector(t, bf16x2);
    t[0] = fmaf((float)((lo >> 8) & 0xffu), s, nzs);   t[1] = fmaf((float)((hi >> 8) & 0xffu), sh, nzs);
    o.p[1] = __builtin_convertvector(t, bf16x2);
    t[0] = fmaf((float)((lo >> 16) & 0xffu), s, nzs);  t[1] = fmaf((float)((hi >> 16) & 0xffu), sh, nzs);
    o.p[2] = __builtin_convertvector(t, bf16x2);
    t[0] = fmaf((float)(lo >> 24), s, nzs);            t[1] = fmaf((float)(hi >> 24), sh, nzs);
    o.p[3] = __builtin_convertvector(t, bf16x2);
    return o.v;
}

// v_permlane32_swap(a, b) returns {[a.low half | b.low half], [a.high half | b.high half]}
// (halves of 32 lanes): `low` is a in lanes 0-31 and b's lanes 0-31 in lanes 32-63; `high` is
// a's lanes 32-63 in lanes 0-31 and b in lanes 32-63.
__device__ inline void swap_halves(uint32_t a, uint32_t b, uint32_t &low, uint32_t &high)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    low = r[0];
    high = r[1];
}

// What one wavefront needs for one step (128 k of its tile): four code vectors, the scale of
// each 32-k unit and the word holding the zero-points of the step's groups.
struct StepRegs {
    uint4 v[4];
    float s[4];
    uint32_t zw;
};

template <int MB, int TN, int KW, bool G128>
__global__ __launch_bounds__(TN * KW * 64) void gemm_small_b4(const GemmArgs A)
{
    constexpr int GEMM_THREADS = TN * KW * 64; // TN tiles x KW k-slices, one wavefront each
    constexpr int ROWS = MB * 32;              // activation rows held (rows past M are zero)
    constexpr int XK = KW * KC;                // k per workgroup iteration
    constexpr int XPITCH = XK + 8;             // bf16 per LDS row: conflict-free 128-bit reads
    constexpr int XLOADS = ROWS * (XK / 4) / GEMM_THREADS;   // float4 loads per thread and chunk
    constexpr int ACC = MB * 2 * 16;           // accumulator registers per lane
    // two activation buffers: the chunk of the next iteration is written while this one is
    // read; reused at the end for the accumulators of the k-slices 1 .. KW-1
    constexpr int XBYTES = 2 * ROWS * XPITCH * 2;
    constexpr int RBYTES = (KW - 1) * TN * ACC * 64 * 4;
    __shared__ __attribute__((aligned(16))) char smem[XBYTES > RBYTES ? XBYTES : RBYTES];
    __bf16 *Xs = (__bf16 *)smem;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tn = wave % TN, kw = wave / TN;
    const int tile = blockIdx.x * TN + tn;
    const bool have_tile = tile < A.tiles;
    const int m0 = blockIdx.z * ROWS;                       // first activation row of this workgroup
    const int rows = A.M - m0 < ROWS ? A.M - m0 : ROWS;      // real rows among the ROWS held
    const int st0 = blockIdx.y * A.steps_per_split;
    int st1 = st0 + A.steps_per_split;
    if (st1 > A.steps) st1 = A.steps;
    const int iters = (st1 - st0 + KW - 1) / KW;

    const int tclamp = have_tile ? tile : A.tiles - 1;
    const uint4 *codes = A.codes + (size_t)tclamp * A.steps * 4 * QG_WAVE + lane;
    const float *sc = A.scales + (size_t)tclamp * A.ngroups * QG_WAVE + lane;
    const uint32_t *zr = A.zeros + (size_t)tclamp * A.zwords * QG_WAVE + lane;

    floatx16 acc[MB][2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mb][nb][i] = 0.0f;

    const int half = lane >> 5;           // which k-octet pair this lane feeds
    const int row = lane & 31;

    // group of unit u (32 k) of a step: G <= 128 has 128/G groups per step, G > 128 has
    // G/128 steps per group (then group_shift is 7 and the unit term vanishes)
    const int step_shift = 7 - A.group_shift;
    auto first_group = [&](int step) { return (step / A.steps_per_group) << step_shift; };
    auto unit_group = [&](int g0, int u) { return g0 + ((u * 32) >> A.group_shift); };
    auto fetch = [&](int step, StepRegs &r) {
#pragma unroll
        for (int u = 0; u < 4; ++u) r.v[u] = codes[((size_t)step * 4 + u) * QG_WAVE];
        const int g0 = first_group(step);
#pragma unroll
        for (int u = 0; u < 4; ++u) r.s[u] = sc[(size_t)unit_group(g0, u) * QG_WAVE];
        r.zw = zr[(size_t)(g0 >> 3) * QG_WAVE];      // a step's groups share one zero word
    };

    // this thread's share of an activation chunk: XLOADS pieces of 4 consecutive k, RPP rows
    // apart, converted to bf16 (round to nearest even) on the way into LDS.  Pieces with no
    // real row are skipped (their LDS rows keep whatever they held), other rows past M repeat
    // the last real row, and k past K repeats the last piece: a row of the A operand only
    // reaches the same row of the result, and rows past M are never stored; k past K belongs
    // to steps no wavefront runs.  Offsets are rebuilt at every use (two operations per piece) rather
    // than kept in registers across the loop.
    constexpr int RPP = GEMM_THREADS / (XK / 4);
    constexpr int XPART = XLOADS / 4;          // pieces issued per 32-k unit of the running step
    const int xrow = threadIdx.x / (XK / 4), xcol = (threadIdx.x % (XK / 4)) * 4;
    float4 xr[XLOADS];
    auto load_x_part = [&](int k0, int part) {
        const float *base = A.X + (size_t)m0 * A.K + k0;     // uniform
        const uint32_t r = opaque((uint32_t)xrow);
        const uint32_t last = (uint32_t)(A.K - 4 - k0);
        const uint32_t col = (uint32_t)xcol < last ? (uint32_t)xcol : last;
#pragma unroll
        for (int j = part * XPART; j < (part + 1) * XPART; ++j) {
            if (j * RPP >= rows) continue;                   // uniform: no real row in this piece
            uint32_t m = r + j * RPP;
            m = m < (uint32_t)rows ? m : (uint32_t)(rows - 1);
            xr[j] = *(const float4 *)(base + (m * (uint32_t)A.K + col));
        }
    };
    auto store_x = [&](int buf) {
        __bf16 *dst = Xs + (size_t)(buf * ROWS + xrow) * XPITCH + xcol;
#pragma unroll
        for (int j = 0; j < XLOADS; ++j) {
            if (j * RPP >= rows) continue;
            floatx2 a = {xr[j].x, xr[j].y}, b = {xr[j].z, xr[j].w};
            bf16x2 pa = __builtin_convertvector(a, bf16x2), pb = __builtin_convertvector(b, bf16x2);
            uint2 packed;
            packed.x = *(uint32_t *)&pa;
            packed.y = *(uint32_t *)&pb;
            *(uint2 *)(dst + j * RPP * XPITCH) = packed;
        }
    };

    // One step of this wavefront: dequantize 64 outputs x 128 k, multiply with all rows.  The
    // A operands of unit u + 1 are read from LDS while unit u is multiplied; with `xk0` >= 0 a
    // quarter of the next activation chunk is requested at the start of every unit, so the
    // memory pipeline works alongside the arithmetic instead of ahead of it.
    auto compute = [&](const StepRegs &r, int step, int buf, int xk0) {
        const int g0 = first_group(step);
        const __bf16 *xs = Xs + (size_t)buf * ROWS * XPITCH + kw * KC + row * XPITCH + half * 16;
        bf16x8 a0[MB], a1[MB], n0[MB], n1[MB];
        uint32_t sP = 0, sQ = 0, nP = 0, nQ = 0;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            a0[mb] = *(const bf16x8 *)(xs + mb * 32 * XPITCH);          // octet 0 or 2
            a1[mb] = *(const bf16x8 *)(xs + mb * 32 * XPITCH + 8);      // octet 1 or 3
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (xk0 >= 0) load_x_part(xk0, u);
            if (u < 3) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    n0[mb] = *(const bf16x8 *)(xs + mb * 32 * XPITCH + (u + 1) * 32);
                    n1[mb] = *(const bf16x8 *)(xs + mb * 32 * XPITCH + (u + 1) * 32 + 8);
                }
            }
            // outputs 0-31 of the tile in both halves (P), outputs 32-63 in both halves (Q);
            // G128: the units of a step share one group, whose scale and zero term are
            // exchanged once per step (the lane exchange costs about five issue slots)
            uint32_t P0, Q0, P1, Q1;
            if (!G128 || u == 0) {
                const float s = r.s[u];
                const int g = unit_group(g0, u);
                const float nzs = -(float)((r.zw >> (4 * (g & 7))) & 15u) * s;
                swap_halves(__float_as_uint(s), __float_as_uint(s), sP, sQ);
                swap_halves(__float_as_uint(nzs), __float_as_uint(nzs), nP, nQ);
            }
            swap_halves(r.v[u].x, r.v[u].z, P0, Q0);   // k-octets 0 (low lanes) and 2 (high lanes)
            swap_halves(r.v[u].y, r.v[u].w, P1, Q1);   // k-octets 1 and 3
            const bf16x8 bP0 = dequant_word(P0, __uint_as_float(sP), __uint_as_float(nP));
            const bf16x8 bQ0 = dequant_word(Q0, __uint_as_float(sQ), __uint_as_float(nQ));
            const bf16x8 bP1 = dequant_word(P1, __uint_as_float(sP), __uint_as_float(nP));
            const bf16x8 bQ1 = dequant_word(Q1, __uint_as_float(sQ), __uint_as_float(nQ));
            // consecutive matrix instructions write different accumulators
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                acc[mb][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[mb], bP0, acc[mb][0], 0, 0, 0);
                acc[mb][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[mb], bQ0, acc[mb][1], 0, 0, 0);
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                acc[mb][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[mb], bP1, acc[mb][0], 0, 0, 0);
                acc[mb][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[mb], bQ1, acc[mb][1], 0, 0, 0);
            }
            if (u < 3) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    a0[mb] = n0[mb];
                    a1[mb] = n1[mb];
                }
            }
            __builtin_amdgcn_sched_barrier(0);     // units stay in order
        }
    };
    // Every iteration but the last has all KW steps inside the split, so the loop body is
    // straight-line code: issue the loads of iteration it + 1, compute iteration it from
    // registers and LDS filled one iteration earlier, then move the new data into place.
    StepRegs cur, nxt;
    if (iters > 0) {
        const int step = st0 + kw;
        fetch(step < st1 ? step : st1 - 1, cur);
#pragma unroll
        for (int part = 0; part < 4; ++part) load_x_part(st0 * KC, part);
        store_x(0);
    }
    __syncthreads();
    int buf = 0;
    for (int it = 0; it + 1 < iters; ++it) {
        const int step = st0 + it * KW + kw;
        const int ns = step + KW;
        fetch(ns < st1 ? ns : st1 - 1, nxt);
        __builtin_amdgcn_sched_barrier(0);     // weight loads first ...
        compute(cur, step, buf, (st0 + (it + 1) * KW) * KC);
        __builtin_amdgcn_sched_barrier(0);     // ... and nothing that waits for them before the arithmetic is done
        store_x(buf ^ 1);
        cur = nxt;
        __syncthreads();      // next chunk written, this chunk's readers done
        buf ^= 1;
    }
    if (iters > 0) {
        const int step = st0 + (iters - 1) * KW + kw;
        if (step < st1) compute(cur, step, buf, -1);
    }

    if constexpr (KW > 1) {
        // k-slices 1 .. KW-1 hand their accumulators to slice 0 of the same tile, which adds
        // them in slice order; the buffers of X are reused once every reader is done
        float *red = (float *)smem;
        __syncthreads();
        if (kw > 0) {
            float *dst = red + ((size_t)((kw - 1) * TN + tn) * ACC) * 64 + lane;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) dst[((mb * 2 + nb) * 16 + i) * 64] = acc[mb][nb][i];
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll
        for (int k = 1; k < KW; ++k) {
            const float *src = red + ((size_t)((k - 1) * TN + tn) * ACC) * 64 + lane;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[mb][nb][i] += src[((mb * 2 + nb) * 16 + i) * 64];
        }
    }

    if (!have_tile) return;
    float *out = A.out + (size_t)blockIdx.y * A.M * A.N;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const int n = tile * QG_WAVE + nb * 32 + row;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int m = m0 + mb * 32 + 8 * (i / 4) + 4 * half + (i % 4);
                if (m < A.M && n < A.N) out[(size_t)m * A.N + n] = acc[mb][nb][i];
            }
        }
}

// ---------------------------------------------------------------------------------------
// The same product for 33 ... 128 rows with every activation row in one wavefront, so each
// weight is dequantized once however many rows there are, and with the dequantization of unit
// u + 1 issued between the matrix instructions of unit u: a wavefront alone keeps the vector
// ALU and the matrix core busy at the same time (the kernel above clumps them, and two
// wavefronts per SIMD that leave a barrier together clump in step).
//
// A workgroup is TN wavefronts = TN neighbouring tiles over the same k range (no k-slices);
// an iteration is a pair of steps (256 k).  The activations of the next pair go through
// registers into the second LDS buffer an eighth at a time, each eighth stored DELAY units
// after it was requested; codes, scales and zero words are requested one iteration (two
// steps) ahead.
// ---------------------------------------------------------------------------------------
template <int MB, int TN, bool G128>
__global__ __launch_bounds__(TN * 64, MB == 2 ? 2 : 1) void gemm_wide_b4(const GemmArgs A)
{
    constexpr int THREADS = TN * 64;
    constexpr int ROWS = MB * 32;
    constexpr int XK = 2 * KC;                              // k per iteration
    constexpr int XPITCH = XK + 8;                          // bf16 per LDS row
    constexpr int XLOADS = ROWS * (XK / 4) / THREADS;       // float4 per thread and chunk
    constexpr int XPART = XLOADS / 8;                       // ... and unit
    constexpr int RPP = THREADS / (XK / 4);                 // rows between a thread's pieces
    constexpr int DELAY = 2;                                // units between a request for activations and its use
    constexpr int NM = MB * 4;                              // matrix instructions per unit
    constexpr int PPM = 16 / NM;                            // pieces of dequantization per matrix instruction
    static_assert(XPART >= 1 && XLOADS % 8 == 0, "a chunk is moved in eight parts");
    static_assert(MB == 2 || MB == 4, "16 pieces are dealt over 8 or 16 matrix instructions");
    __shared__ __attribute__((aligned(16))) char smem[2 * ROWS * XPITCH * 2];
    __bf16 *Xs = (__bf16 *)smem;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x * TN + wave;
    const bool have_tile = tile < A.tiles;
    const int rows = A.M < ROWS ? A.M : ROWS;
    const int st0 = blockIdx.y * A.steps_per_split;
    int st1 = st0 + A.steps_per_split;
    if (st1 > A.steps) st1 = A.steps;
    const int npairs = (st1 - st0 + 1) / 2;

    const int tclamp = have_tile ? tile : A.tiles - 1;
    const uint4 *codes = A.codes + (size_t)tclamp * A.steps * 4 * QG_WAVE + lane;
    const float *sc = A.scales + (size_t)tclamp * A.ngroups * QG_WAVE + lane;
    const uint32_t *zr = A.zeros + (size_t)tclamp * A.zwords * QG_WAVE + lane;

    floatx16 acc[MB][2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mb][nb][i] = 0.0f;

    const int half = lane >> 5;
    const int row = lane & 31;
    const int step_shift = 7 - A.group_shift;
    auto first_group = [&](int step) { return (step / A.steps_per_group) << step_shift; };
    auto unit_group = [&](int g0, int u) { return g0 + ((u * 32) >> A.group_shift); };
    auto fetch = [&](int step, StepRegs &r) {
        step = step < st1 ? step : st1 - 1;            // past the range: loaded again, not used
#pragma unroll
        for (int u = 0; u < 4; ++u) r.v[u] = codes[((size_t)step * 4 + u) * QG_WAVE];
        const int g0 = first_group(step);
#pragma unroll
        for (int u = 0; u < 4; ++u) r.s[u] = sc[(size_t)unit_group(g0, u) * QG_WAVE];
        r.zw = zr[(size_t)(g0 >> 3) * QG_WAVE];
    };

    // Activations: piece j of a thread is 4 consecutive k of row j * RPP + wave, so a wavefront
    // reads 1 KB of one row.  Rows past M repeat the last real row (a row of the A operand only
    // reaches the same row of the result, and those are not stored); k past K repeats the last
    // piece of the row (it belongs to a step that is not run).  No branches: the loads of a
    // part must stay countable for the waits that follow.
    const int xcol = lane * 4;
    auto load_x = [&](int k0, int j, float4 &dst) {
        const float *base = A.X + k0;                          // uniform
        const uint32_t last = (uint32_t)(A.K - 4 - k0);
        const uint32_t col = (uint32_t)xcol < last ? (uint32_t)xcol : last;
        int m = j * RPP + wave;                                // uniform
        m = m < rows ? m : rows - 1;
        dst = *(const float4 *)(base + ((size_t)m * (uint32_t)A.K + col));
    };
    auto store_x = [&](int buf, int j, const float4 &src) {
        floatx2 a = {src.x, src.y}, b = {src.z, src.w};
        bf16x2 pa = __builtin_convertvector(a, bf16x2), pb = __builtin_convertvector(b, bf16x2);
        uint2 packed;
        packed.x = *(uint32_t *)&pa;
        packed.y = *(uint32_t *)&pb;
        *(uint2 *)(Xs + (size_t)(buf * ROWS + j * RPP + wave) * XPITCH + xcol) = packed;
    };

    // Dequantization of one unit in 16 pieces (4 words x 4 byte positions, two codes each).
    struct UnitPrep {
        uint32_t lo[4], hi[4];     // words P0, Q0, P1, Q1: even codes, odd codes (times 16)
        float s[2], sh[2], nz[2];  // of outputs 0-31 (P) and 32-63 (Q)
    };
    // G128: the four units of a step share one group (G >= 128), so the scale and zero term
    // are exchanged between the halves once per step (the lane exchange is the most expensive
    // vector instruction of the loop: about five issue slots)
    auto prepare = [&](const StepRegs &r, int g0, int u, UnitPrep &pr) {
        uint32_t w[4];
        if (!G128 || u == 0) {
            const float s = r.s[u];
            const int g = unit_group(g0, u);
            const float nzs = -(float)((r.zw >> (4 * (g & 7))) & 15u) * s;
            uint32_t sP, sQ, nP, nQ;
            swap_halves(__float_as_uint(s), __float_as_uint(s), sP, sQ);
            swap_halves(__float_as_uint(nzs), __float_as_uint(nzs), nP, nQ);
            pr.s[0] = __uint_as_float(sP);  pr.s[1] = __uint_as_float(sQ);
            pr.sh[0] = pr.s[0] * 0.0625f;   pr.sh[1] = pr.s[1] * 0.0625f;
            pr.nz[0] = __uint_as_float(nP); pr.nz[1] = __uint_as_float(nQ);
        }
        swap_halves(r.v[u].x, r.v[u].z, w[0], w[1]);       // k-octets 0 | 2
        swap_halves(r.v[u].y, r.v[u].w, w[2], w[3]);       // k-octets 1 | 3
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pr.lo[i] = opaque(w[i] & 0x0f0f0f0fu);
            pr.hi[i] = opaque(w[i] & 0xf0f0f0f0u);
        }
    };
    UnitPrep pr;               // lives across units and iterations: with G128 its scale part is per step
    auto piece = [&](const UnitPrep &pr, int i, Operand (&o)[4]) {
        const int wd = i >> 2, j = i & 3, pq = wd & 1;
        floatx2 t;
        t[0] = fmaf((float)((pr.lo[wd] >> (8 * j)) & 0xffu), pr.s[pq], pr.nz[pq]);
        t[1] = fmaf((float)((pr.hi[wd] >> (8 * j)) & 0xffu), pr.sh[pq], pr.nz[pq]);
        bf16x2 pair = __builtin_convertvector(t, bf16x2);
        // an empty volatile statement: keeps this piece in the slot it is written in
        uint32_t bits = *(uint32_t *)&pair;
        asm volatile("" : "+v"(bits));
        o[wd].p[j] = *(bf16x2 *)&bits;
    };

    // The units of one iteration.  Matrix instruction k of unit uu is followed by pieces of
    // the dequantization of unit uu + 1 (of the next pair's first step after the last unit,
    // if NEXT), by the LDS reads of that unit's A operands and by the traffic of the next
    // activation chunk; every such slot is fenced, so the order written here is the order
    // issued.  bq: B operands P0, Q0, P1, Q1 of the unit about to be multiplied.
    auto compute = [&](auto nu_tag, auto next_tag, const StepRegs &r0, const StepRegs &r1, const StepRegs &rn,
                       int step0, int buf, Operand (&bq)[4]) {
        constexpr int NU = decltype(nu_tag)::value;
        constexpr bool NEXT = decltype(next_tag)::value;
        const int g00 = first_group(step0), g01 = first_group(step0 + 1), g02 = first_group(step0 + 2);
        const int xk0 = (step0 + 2) * KC;
        const __bf16 *xs = Xs + (size_t)buf * ROWS * XPITCH + row * XPITCH + half * 16;
        bf16x8 a0[MB], a1[MB], n0[MB], n1[MB];
        float4 xr[DELAY + 1][XPART];
        Operand bn[4];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            a0[mb] = *(const bf16x8 *)(xs + mb * 32 * XPITCH);
            a1[mb] = *(const bf16x8 *)(xs + mb * 32 * XPITCH + 8);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int uu = 0; uu < NU; ++uu) {
            const bool more = uu + 1 < NU;                  // next unit in this pair
            const bool dq = more || NEXT;                   // something to dequantize
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                const int mb = (k % (MB * 2)) / 2, nb = k % 2;
                if (k < MB * 2)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[mb], bq[nb].v, acc[mb][nb], 0, 0, 0);
                else
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[mb], bq[2 + nb].v, acc[mb][nb], 0, 0, 0);
                if (k == 0) {
                    if (NEXT) {
#pragma unroll
                        for (int i = 0; i < XPART; ++i) load_x(xk0, uu * XPART + i, xr[uu % (DELAY + 1)][i]);
                    }
                    if (more) {
#pragma unroll
                        for (int m2 = 0; m2 < MB; ++m2) {
                            n0[m2] = *(const bf16x8 *)(xs + m2 * 32 * XPITCH + (uu + 1) * 32);
                            n1[m2] = *(const bf16x8 *)(xs + m2 * 32 * XPITCH + (uu + 1) * 32 + 8);
                        }
                    }
                    if (dq) {
                        if (more) prepare(uu + 1 < 4 ? r0 : r1, uu + 1 < 4 ? g00 : g01, (uu + 1) & 3, pr);
                        else prepare(rn, g02, 0, pr);
                    }
                }
                if (dq) {
#pragma unroll
                    for (int q = 0; q < PPM; ++q) piece(pr, k * PPM + q, bn);
                }
                if (NEXT && k == NM / 2 && uu >= DELAY) {
#pragma unroll
                    for (int i = 0; i < XPART; ++i)
                        store_x(buf ^ 1, (uu - DELAY) * XPART + i, xr[(uu - DELAY) % (DELAY + 1)][i]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (more) {
#pragma unroll
                for (int m2 = 0; m2 < MB; ++m2) {
                    a0[m2] = n0[m2];
                    a1[m2] = n1[m2];
                }
            }
            if (dq) {
#pragma unroll
                for (int i = 0; i < 4; ++i) bq[i].v = bn[i].v;
            }
        }
        if (NEXT) {
#pragma unroll
            for (int uu = NU - DELAY; uu < NU; ++uu)
#pragma unroll
                for (int i = 0; i < XPART; ++i) store_x(buf ^ 1, uu * XPART + i, xr[uu % (DELAY + 1)][i]);
        }
    };

    using std::integral_constant;
    StepRegs c0, c1, n0, n1;
    Operand bq[4];
    if (npairs > 0) {
        fetch(st0, c0);
        fetch(st0 + 1, c1);
        float4 xall[XLOADS];
#pragma unroll
        for (int j = 0; j < XLOADS; ++j) load_x(st0 * KC, j, xall[j]);
#pragma unroll
        for (int j = 0; j < XLOADS; ++j) store_x(0, j, xall[j]);
        prepare(c0, first_group(st0), 0, pr);
#pragma unroll
        for (int i = 0; i < 16; ++i) piece(pr, i, bq);
    }
    __syncthreads();
    int buf = 0;
    for (int p = 0; p + 1 < npairs; ++p) {
        const int s = st0 + 2 * p;
        fetch(s + 2, n0);
        fetch(s + 3, n1);
        __builtin_amdgcn_sched_barrier(0);
        compute(integral_constant<int, 8>(), integral_constant<bool, true>(), c0, c1, n0, s, buf, bq);
        __builtin_amdgcn_sched_barrier(0);
        c0 = n0;
        c1 = n1;
        __syncthreads();      // next chunk written, this chunk's readers done
        buf ^= 1;
    }
    if (npairs > 0) {
        const int s = st0 + 2 * (npairs - 1);
        if (s + 1 < st1) compute(integral_constant<int, 8>(), integral_constant<bool, false>(), c0, c1, c1, s, buf, bq);
        else compute(integral_constant<int, 4>(), integral_constant<bool, false>(), c0, c1, c1, s, buf, bq);
    }

    if (!have_tile) return;
    float *out = A.out + (size_t)blockIdx.y * A.M * A.N;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const int n = tile * QG_WAVE + nb * 32 + row;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int m = mb * 32 + 8 * (i / 4) + 4 * half + (i % 4);
                if (m < A.M && n < A.N) out[(size_t)m * A.N + n] = acc[mb][nb][i];
            }
        }
}


// Y = sum of the K-split partial results, in split order.  All (up to 8) loads of a thread
// are issued before the first addition; a loop over a run-time split count would wait for
// each load in turn.
__global__ void add_splits(const float *__restrict__ partial, int splits, size_t count,
                           float *__restrict__ Y)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    float v[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = s < splits ? partial[(size_t)s * count + i] : 0.0f;
    float t = v[0];
#pragma unroll
    for (int s = 1; s < 8; ++s) t += v[s];       // the missing ones add +0.0
    Y[i] = t;
}

// The same for the raw-code kernel (parts as it writes them: quads of 4 rows x 32 outputs, lane = row half and
// output).  A block of outputs and rows has `ranges` parts or, with ranges == 0, as many as workgroups its
// units fell to (one: that workgroup has stored Y itself).  A workgroup is one wavefront of W elements per lane.
// What bounds it is the way of the parts from the other dies, so as long as the chip has room the more wavefronts
// ask at once the better; two elements per lane keep whole lines of Y together.  A call with eight parts, us, with
// four elements per lane and four wavefronts per workgroup | two | one: 2048 x 2048 M = 24 10.1 | 10.2 | 9.3, 4096 x 4096
// M = 24 11.5 | 11.0 | 10.8, M = 128 23.5 | 22.2 | 22.5, 8192 x 8192 M = 128 32.0 | 30.6 | 31.6.
template <int W>
__global__ __launch_bounds__(64) void add_parts(const char *__restrict__ partial, int tiles, int N, int M, int tn, int rows,
                                                int zblocks, int units, int ranges, int quota, float *__restrict__ Y)
{
    typedef float vec __attribute__((ext_vector_type(W)));
    constexpr int WAVES = 4 / W;                              // per quad
    const int bands = (M + 7) / 8;
    const int q = blockIdx.x / WAVES;                         // (tile, band, pq)
    const int at = (blockIdx.x % WAVES * 64 + threadIdx.x) * W;       // element of the quad
    const int pq = q & 1, band = (q >> 1) % bands, tile = (q >> 1) / bands;
    int count = ranges;
    if (ranges == 0) {
        const int b = tile / tn * zblocks + band * 8 / rows;
        count = ((b + 1) * units - 1) / quota - b * units / quota + 1;
        if (count == 1) return;
    }
    vec v[QG_MAX_SEGMENTS];
#pragma unroll
    for (int s = 0; s < QG_MAX_SEGMENTS; ++s)
        v[s] = s < count ? *(const vec *)(partial + (((size_t)s * tiles + tile) * bands + band) * 2048 + pq * 1024 + at * 4) : (vec)0.0f;
    vec t = v[0];
#pragma unroll
    for (int s = 1; s < QG_MAX_SEGMENTS; ++s) t += v[s];      // the missing ones add +0.0
    const int lane = at / 4, n = tile * QG_WAVE + 32 * pq + (lane & 31), m = band * 8 + 4 * (lane >> 5) + at % 4;
    if (n >= N) return;
#pragma unroll
    for (int j = 0; j < W; ++j)
        if (m + j < M) Y[(size_t)(m + j) * N + n] = t[j];
}

bool fast_path(const QgLayout &L)
{
    return L.bits == 4 && L.group % 32 == 0 && L.K % KC == 0 && L.K <= (1 << 20) &&
           (L.group <= KC ? KC % L.group == 0 : L.group % KC == 0);
}

int g_tune_splits = 0;      // measurement knobs: 0 = built-in choice
int g_tune_shape = 0;       // 1 + index into SHAPES, NSHAPES + 1: the raw-code kernel, -1: gemm_rows16

// Choices recorded per problem (qg_gemm_autotune): used where both knobs are 0.
struct GemmTuneEntry {
    int64_t N, K;
    int bits, group, M, splits, shape;
};
constexpr int GEMM_TUNE_ENTRIES = 64;
GemmTuneEntry g_gemm_table[GEMM_TUNE_ENTRIES];
int g_gemm_count = 0, g_gemm_next = 0;
std::mutex g_gemm_mutex;

bool gemm_tuning_for(int64_t N, int64_t K, int bits, int group, int M, int *splits, int *shape)
{
    std::lock_guard<std::mutex> lock(g_gemm_mutex);
    for (int i = 0; i < g_gemm_count; ++i) {
        const GemmTuneEntry &e = g_gemm_table[i];
        if (e.N == N && e.K == K && e.bits == bits && e.group == group && e.M == M) {
            *splits = e.splits;
            *shape = e.shape;
            return true;
        }
    }
    return false;
}

void gemm_record_tuning(int64_t N, int64_t K, int bits, int group, int M, int splits, int shape)
{
    std::lock_guard<std::mutex> lock(g_gemm_mutex);
    int at = -1;
    for (int i = 0; i < g_gemm_count; ++i) {
        const GemmTuneEntry &e = g_gemm_table[i];
        if (e.N == N && e.K == K && e.bits == bits && e.group == group && e.M == M) at = i;
    }
    if (at < 0) {
        if (g_gemm_count < GEMM_TUNE_ENTRIES) at = g_gemm_count++;
        else { at = g_gemm_next; g_gemm_next = (g_gemm_next + 1) % GEMM_TUNE_ENTRIES; }
    }
    g_gemm_table[at] = {N, K, bits, group, M, splits, shape};
}

int gcd(int a, int b) { return b == 0 ? a : gcd(b, a % b); }

using KernelInfo = QgKernelInfo;

template <int MB, int TN, int KW>
void launch(const GemmArgs &A, dim3 grid, hipStream_t st, KernelInfo *query)
{
    if (query) {
        *query = {A.group_shift == 7 ? (const void *)gemm_small_b4<MB, TN, KW, true>
                                     : (const void *)gemm_small_b4<MB, TN, KW, false>, TN * KW * 64, 0};
        return;
    }
    if (A.group_shift == 7)
        hipLaunchKernelGGL((gemm_small_b4<MB, TN, KW, true>), grid, dim3(TN * KW * 64), 0, st, A);
    else
        hipLaunchKernelGGL((gemm_small_b4<MB, TN, KW, false>), grid, dim3(TN * KW * 64), 0, st, A);
}

template <int MB, int TN>
void launch_wide(const GemmArgs &A, dim3 grid, hipStream_t st, KernelInfo *query)
{
    if (query) {
        *query = {A.group_shift == 7 ? (const void *)gemm_wide_b4<MB, TN, true> : (const void *)gemm_wide_b4<MB, TN, false>,
                  TN * 64, 0};
        return;
    }
    if (A.group_shift == 7) hipLaunchKernelGGL((gemm_wide_b4<MB, TN, true>), grid, dim3(TN * 64), 0, st, A);
    else hipLaunchKernelGGL((gemm_wide_b4<MB, TN, false>), grid, dim3(TN * 64), 0, st, A);
}

// Workgroup shapes: {rows / 32, tiles, k-slices, gemm_wide_b4 (all rows in one wavefront)}
struct Shape {
    int mb, tn, kw;
    bool wide;
};
constexpr Shape SHAPES[] = {
    {1, 1, 4, false}, {1, 2, 4, false}, {1, 4, 2, false},                       // up to 32 rows
    {2, 2, 2, false}, {2, 4, 1, false}, {2, 4, 2, false}, {2, 8, 1, false},     // blocks of 64 rows
    {2, 4, 1, true},  {2, 2, 1, true},                                          // up to 64 rows
    {4, 4, 1, true},  {4, 2, 1, true},                                          // up to 128 rows
    {2, 8, 1, true},                                                            // up to 64 rows
};
constexpr int NSHAPES = sizeof(SHAPES) / sizeof(SHAPES[0]);

void launch_shape(int i, const GemmArgs &A, dim3 grid, hipStream_t st, KernelInfo *query = nullptr)
{
    switch (i) {
    case 0: launch<1, 1, 4>(A, grid, st, query); break;
    case 1: launch<1, 2, 4>(A, grid, st, query); break;
    case 2: launch<1, 4, 2>(A, grid, st, query); break;
    case 3: launch<2, 2, 2>(A, grid, st, query); break;
    case 4: launch<2, 4, 1>(A, grid, st, query); break;
    case 5: launch<2, 4, 2>(A, grid, st, query); break;
    case 6: launch<2, 8, 1>(A, grid, st, query); break;
    case 7: launch_wide<2, 4>(A, grid, st, query); break;
    case 8: launch_wide<2, 2>(A, grid, st, query); break;
    case 9: launch_wide<4, 4>(A, grid, st, query); break;
    case 10: launch_wide<4, 2>(A, grid, st, query); break;
    default: launch_wide<2, 8>(A, grid, st, query); break;
    }
}


// ---- gemm_codes: which layouts it takes, and its launch ----
// (X is rounded to bf16 on this path.  Layouts outside it keep an fp32 product, also where the kernel could take
// them: 3-bit groups of 32, 2- and 3-bit groups of an odd number of 128 k.)
int codes_gps(const QgLayout &L)       // groups per step of 128 k, 0: groups of several steps, -1: not taken
{
    if (L.K % 16 != 0 || L.K > (1 << 22)) return -1;
    if (L.group > KC) return L.group % (L.unit * L.step_units) == 0 ? 0 : -1;
    const int least = L.bits == 4 ? 16 : L.bits == 2 ? 32 : 64;
    return L.group >= least && KC % L.group == 0 ? KC / L.group : -1;
}

// Workspace of the raw-code path: A operands, counters, partial results of the K ranges.
struct CodesSpace {
    size_t arrived_off, partial_off, total;
    int rows_padded, steps_padded, groupk;
};
CodesSpace codes_space(const QgLayout &L, int gps, int M)
{
    CodesSpace W;
    const int rows_per_block = M <= 32 ? 32 : 64;
    W.rows_padded = (M + rows_per_block - 1) / rows_per_block * rows_per_block;
    W.steps_padded = (int)((L.K + 4 * KC - 1) / (4 * KC) * 4);
    W.groupk = L.group > KC ? KC : L.group;
    W.arrived_off = (size_t)W.rows_padded / 32 * W.steps_padded * qg_codes_seq(gps) * 1024;
    W.partial_off = qg_round_up(W.arrived_off + (size_t)L.tiles * 4 * sizeof(uint32_t), QG_SECTION_ALIGN);
    W.total = qg_round_up(W.partial_off + (size_t)QG_MAX_SEGMENTS * L.tiles * ((M + 7) / 8) * 2048, QG_SECTION_ALIGN);
    return W;
}

// How a raw-code product is cut: workgroups of TN tiles x KW k-slices, MB blocks of 32 rows; units of KW
// steps; `ranges` K ranges per block of outputs and rows (one workgroup each), or, with ranges == 0,
// `quota` consecutive units per workgroup whatever blocks they fall into.
struct CodesPlan {
    int mb, tn, kw, zblocks, blocks, units, ranges, quota, workgroups, parts;
    bool fused, self;
    int kernels;               // of a call
    double us, kernels_us;     // what it costs, and what its kernels take of that (codes_price)
    double cut_us;             // ... as blocks of 64 rows are cut by (codes_cut_us)
};

// Cuts into at most `most` parts per block, one workgroup per compute unit at most where that is possible (a
// workgroup takes half of a unit's registers or more, so one more would wait for a second round): whole ranges
// of K, or, where more workgroups than `room` per block would be needed for them, `even` units per workgroup.
void codes_cut(CodesPlan &P, int most, int room, int even)
{
    int ranges = room < most ? room : most;
    if (ranges < 1) ranges = 1;
    if (ranges > P.units) ranges = P.units;
    P.quota = (P.units + ranges - 1) / ranges;
    P.ranges = P.parts = (P.units + P.quota - 1) / P.quota;
    P.workgroups = P.blocks * P.ranges;
    if (most <= room || even >= P.quota) return;
    const int parts = (P.units + even - 2) / even + 1;          // of a block that begins at the end of a quota
    if (parts <= most) {
        P.quota = even;
        P.ranges = 0;
        P.parts = parts;
        P.workgroups = (P.blocks * P.units + even - 1) / even;
    }
}

// Estimate of a call: straight lines through measured cuts of 2, 3 and 4 bits, groups of 16, 32, 64, 128 and one
// per output.  Up to 32 rows: 9000 cuts of 18 matrices from 512 x 512 to 30000 x 4096 (root mean square of what it is
// off: 4 %); more: 10000 cuts of 29 matrices, with blocks of 32 rows (5 %) and of 64 (4 %).  A unit has a time of its
// own, by rows and groups per step, and one on a full chip for the weights it reads.
// Parts are added by a kernel, which the whole chip shares, or, if they are two or three, by the workgroup that
// comes last, which alone reads them all: at 32 rows that is never the slower way, at 64 from 8 MB of
// parts (two of them) or 11 (three) on (kernel minus last workgroup, us: -3 below 2 MB, +2 at 12 MB of two
// parts).  An evenly dealt workgroup ends a block of outputs in the middle of its units as well as at their end.
// (A table that went by the groups per step alone and took the adding for 1 us at two parts put 5120 x 5120 3-bit g64
// M = 16 on 80 workgroups, 14.0 -> 15.3 us, and 4096 x 4096 3-bit M = 8 on 64, 10.6 -> 13.0; now 11.9 and 10.3.)
struct CodesCost {
    double call, unit, weights;        // of a call, of a unit, of a unit on a full chip for its weights
    double dealt;                      // of a call whose units are dealt evenly
    double last, last_mb, kernel, kernel_mb;       // adding, by the last workgroup and by a kernel, per MB of parts
    double last_workgroup, last_workgroup_mb, part_mb;      // (who adds: the last workgroup against 1.5 + 0.5 per MB)
    double cut_unit, cut_weights;      // (codes_cut_us)
    double self_call, self_unit, self_weights, self_dealt, self_round, self_y_mb, self_kernel, self_kernel_mb;     // (codes_self_us; 0: not taken)
    int cus;
    bool by_parts;                     // the last workgroup's time per MB grows with the parts
};
CodesCost codes_cost(const QgLayout &L, int gps, int M, int mb, int cus, bool self)
{
    static constexpr double SELF_US[2][4] = {{1.14, 1.17, 1.33, 1.64}, {1.80, 1.85, 2.07, 2.46}};
    static constexpr double UNIT_US[3][5] = {{1.0, 1.05, 1.2, 1.45, 2.0}, {1.0, 1.02, 1.18, 1.45, 2.0}, {1.36, 1.38, 1.65, 2.15, 3.2}};
    static constexpr double CUT_UNIT_US[5] = {1.35, 1.4, 1.65, 2.15, 3.2};
    CodesCost C;
    C.part_mb = 4e-6 * M * (double)L.N;
    C.cus = cus;
    C.by_parts = mb == 2;
    C.last_workgroup = mb == 1 ? 1.5 : 4.6;
    C.last_workgroup_mb = mb == 1 ? 0.3 : 0.1;
    C.unit = UNIT_US[M <= 32 ? 0 : mb][gps == 0 ? 0 : gps == 1 ? 1 : gps == 2 ? 2 : gps == 4 ? 3 : 4];
    C.cut_unit = CUT_UNIT_US[gps == 0 ? 0 : gps == 1 ? 1 : gps == 2 ? 2 : gps == 4 ? 3 : 4];
    C.cut_weights = L.bits == 4 ? 0.5 : L.bits == 3 ? 0.35 : 0.1;
    C.self_call = 0.0;
    if (self && mb == 1 && gps <= 4) {
        C.self_unit = SELF_US[M <= 32 ? 0 : 1][gps == 4 ? 3 : gps];
        if (M <= 32) {
            C.self_call = 3.7;
            C.self_unit += M > 16 ? 0.55 : 0.0;
            C.self_weights = L.bits == 4 ? 0.31 : L.bits == 3 ? 0.28 : 0.0;
            C.self_dealt = 2.0, C.self_round = 0.0;
            C.self_y_mb = 0.24, C.self_kernel = 1.7, C.self_kernel_mb = 0.44;
        } else {
            C.self_call = 3.6, C.self_weights = 0.0;
            C.self_dealt = 0.0, C.self_round = 1.9;
            C.self_y_mb = 0.12, C.self_kernel = 1.3, C.self_kernel_mb = 0.8;
        }
    }
    if (M <= 32) {
        C.call = 6.0;
        C.weights = L.bits == 4 ? 0.5 : L.bits == 3 ? 0.35 : 0.1;
        C.dealt = 1.4;
        C.last = 1.5, C.last_mb = 0.3, C.kernel = 1.5, C.kernel_mb = 0.5;
        return C;
    }
    // (32 rows of X converted, and Y written)
    const double converted = 1e-5 * ((M + 31) / 32) * (double)L.K;
    C.call = mb == 1 ? 7.3 + 6.3 * converted + 0.26 * C.part_mb : 7.7 + 3.0 * converted + 0.16 * C.part_mb;
    C.weights = L.bits == 4 ? (mb == 1 ? 0.3 : 0.28) : L.bits == 3 ? 0.14 : 0.0;
    C.dealt = 0.0;
    C.last = mb == 1 ? 1.65 : 3.7, C.last_mb = mb == 1 ? 0.06 : 0.3;
    C.kernel = mb == 1 ? 1.4 : 1.7, C.kernel_mb = mb == 1 ? 0.55 : 0.42;
    return C;
}
// What a call takes of the caller's time, whatever its kernels take: a launch is 2.1 us of it, a problem of a launch 0.03.
// A call is priced at the longer of the two, and a fifth of its kernels' time: of calls that all wait for the caller the
// one with the shorter kernels is there first.
double call_us(double kernels_us, int launches, int problems = 0)
{
    const double host = 2.9 + 2.1 * launches + 0.03 * problems;
    return (kernels_us > host ? kernels_us : host) + 0.2 * kernels_us;
}
// Blocks of 32 rows that make their A operands themselves (gemm_codes, SELF): no prepare_x, but every block of
// outputs converts X again, so a unit takes longer, hardly so up to 16 rows.  Lines through 1600 cuts of 400 random
// products of 2 ... 32 rows (2.5 % off) and 1100 of 33 ... 128 (2.9 %).
double codes_self_us(const CodesPlan &P, const CodesCost &C)
{
    const int rounds = (P.workgroups + C.cus - 1) / C.cus;
    const double full = P.workgroups < C.cus ? (double)P.workgroups / C.cus : 1.0;
    double us = C.self_call + P.quota * rounds * (C.self_unit + C.self_weights * full) + C.self_round * (rounds - 1) + C.self_y_mb * C.part_mb;
    if (P.ranges == 0) us += C.self_dealt;
    if (P.parts > 1) us += C.self_kernel + C.self_kernel_mb * P.parts * C.part_mb;
    return us;
}
constexpr double CODES_LEAST_US = 4.8;       // what no plan's kernels are priced below
// Sets P.us, P.kernels_us and, with them, who makes the A operands and who adds the parts.
void codes_price(CodesPlan &P, const CodesCost &C)
{
    P.us = C.call;
    if (P.workgroups <= C.cus) {
        P.us += P.quota * (C.unit + C.weights * P.workgroups / C.cus);
    } else {
        P.us += (P.workgroups + C.cus - 1) / C.cus * P.quota * (C.unit + C.weights);
    }
    if (P.ranges == 0) P.us += C.dealt;
    P.fused = P.self = false;
    if (P.parts > 1) {
        const double mb = P.parts * C.part_mb;
        if (P.parts <= QG_FUSED_SEGMENTS)
            P.fused = C.last_workgroup + C.last_workgroup_mb * (C.by_parts ? P.parts - 1 : 1) * mb <= 1.5 + 0.5 * mb;
        P.us += P.fused ? C.last + C.last_mb * mb : C.kernel + C.kernel_mb * mb;
    }
    P.kernels = P.parts > 1 && !P.fused ? 3 : 2;
    P.kernels_us = P.us;
    P.us = call_us(P.us, P.kernels);
    if (C.self_call > 0.0) {
        const int kernels = P.parts > 1 ? 2 : 1;
        const double kernels_us = codes_self_us(P, C), us = call_us(kernels_us, kernels);
        if (us < P.us) {
            P.us = us;
            P.kernels_us = kernels_us;
            P.kernels = kernels;
            P.self = true;
            P.fused = false;
        }
    }
}

// By which the cuts of blocks of 64 rows are compared: the line fitted through cuts of 2 ... 128 rows.  (The one above, through
// cuts of more than 32 rows, tells blocks of 32 from blocks of 64, but takes dealt units for 10 to 16 % less than they
// need on a long K: 14611 x 6784 2-bit M = 70 34.3 us for 39.1 in dealt units, 36.0 as cut here; 7614 x 20608 3-bit M = 90 52.6
// for 62.8, 58.2.)
double codes_cut_us(const CodesPlan &P, const CodesCost &C)
{
    const int rounds = (P.workgroups + C.cus - 1) / C.cus;
    double us = rounds * P.quota * (C.cut_unit + C.cut_weights * (rounds > 1 ? 1.0 : (double)P.workgroups / C.cus));
    if (P.ranges == 0) us += 1.4;
    const double mb = P.parts * C.part_mb;
    if (P.parts > 1) us += P.fused ? C.last_workgroup + C.last_workgroup_mb * (P.parts - 1) * mb : 1.5 + 0.5 * mb;
    return us;
}

// The best of the cuts into at most 1 ... 8 parts by what they cost; a forced count (the search's, too) takes the one cut.
// A count that would need more workgroups than compute units is dealt evenly over those.
CodesPlan codes_plan_rows(const QgLayout &L, int gps, int M, int mb, int knob_splits, bool by_number)
{
    CodesPlan P;
    P.mb = mb;
    P.zblocks = (M + 32 * mb - 1) / (32 * mb);
    const int cus = qg_compute_units();
    P.kw = qg_codes_kw(gps, P.mb, (L.tiles + 3) / 4 * QG_MAX_SEGMENTS >= cus);
    P.tn = 8 / P.kw;
    P.blocks = (int)((L.tiles + P.tn - 1) / P.tn) * P.zblocks;
    P.units = (int)(((L.K + KC - 1) / KC + P.kw - 1) / P.kw);
    const CodesCost cost = codes_cost(L, gps, M, P.mb, cus, !by_number);
    const int room = cus / P.blocks > 1 ? cus / P.blocks : 1;
    // (several blocks of 32 rows: whole ranges alone, dealt ones no longer share a tile's weights: 8192 x 22016 4-bit
    // M = 72 115 us against 74 in blocks of 64)
    const int even = mb == 1 && P.zblocks > 1 ? 1 << 30 : (int)(((int64_t)P.blocks * P.units + cus - 1) / cus);
    if (knob_splits) {
        codes_cut(P, knob_splits, room, even);
        codes_price(P, cost);
        return P;
    }
    CodesPlan best = P, last = P;
    last.quota = last.ranges = -1;
    for (int most = 1; most <= QG_MAX_SEGMENTS && most <= P.units; ++most) {
        CodesPlan c = P;
        codes_cut(c, most, room, even);
        if (c.quota == last.quota && c.ranges == last.ranges) continue;        // (priced already)
        codes_price(c, cost);
        if (mb == 2) c.cut_us = codes_cut_us(c, cost);
        if (most == 1 || (mb == 2 ? c.cut_us < best.cut_us : c.us < best.us)) best = c;
        last = c;
    }
    return best;
}

// More than 32 rows: in blocks of 64, or of 32 where their price is lower.  A block of 64 unpacks a weight once for
// all of its rows, 1.35 us a unit; a workgroup of blocks of 32 takes half the tiles and twice the k-slices in 1.0 us, so K is
// cut into a quarter of the parts, which is more wherever tiles are few.  us per call, blocks of 64 | 32: 5120 x 5120 2-bit
// g32 M = 48 20.1 | 16.3, 4096 x 4096 3-bit g64 M = 64 17.0 | 13.3, 13824 x 5120 3-bit g64 M = 37 21.5 | 20.6; 22016 x 8192
// 2-bit g32 M = 128 76 | 90.  Over 504 products of 33 ... 128 rows at 2 and 3 bits the choice takes 0.90 of the time of
// blocks of 64 alone, the best cut of either kind 0.88.  (All on weights that the last-level cache holds.  From memory blocks of 32 lose
// more, 13824 x 5120 M = 37 23.2 | 24.8, 4096 x 11008 4-bit M = 128 27.2 | 30.0; the choice then takes 0.90 over 120 products.  Where the
// prices are within 3 % of each other either kind is the faster one, 0.88 ... 1.08.)
// A forced count on the kernel asked for by number (shape 13) keeps blocks of 64, and that kernel's operands come
// from prepare_x.
CodesPlan codes_plan(const QgLayout &L, int gps, int M, int knob_splits, bool by_number)
{
    if (M <= 32) return codes_plan_rows(L, gps, M, 1, knob_splits, by_number);
    const CodesPlan two = codes_plan_rows(L, gps, M, 2, knob_splits, by_number);
    if (knob_splits && by_number) return two;
    const CodesPlan one = codes_plan_rows(L, gps, M, 1, knob_splits, by_number);
    return one.us < two.us ? one : two;
}
}  // namespace

// What a call takes at least.
static size_t gemm_workspace_least(const QgLayout &L, int M)
{
    // partial results of the K split, or the GEMV workspaces of the rows of one grouped launch
    const size_t partial = (size_t)MAX_SPLITS * M * L.N * sizeof(float);
    const size_t gemv = qg_round_up((size_t)L.tiles * (QG_MAX_CHUNKS + 1) * QG_WAVE * sizeof(uint32_t),
                                    QG_SECTION_ALIGN);                                    // as qg_gemv asks
    const int rows = M < QG_MAX_GROUPED ? M : QG_MAX_GROUPED;
    size_t need = fast_path(L) && partial > gemv * rows ? partial : gemv * rows;
    const int gps = codes_gps(L);
    if (M > 1 && gps >= 0 && codes_space(L, gps, M).total > need) need = codes_space(L, gps, M).total;
    return qg_round_up(need, QG_SECTION_ALIGN);
}
// (3-bit groups of 32: the int8 product's operands and parts lie behind the meeting slots of the products per row, which
// stay as qg_workspace_init has left them: behind those of as many rows as a launch takes, whatever the call's M, so that
// a buffer large enough for several M serves them in any order)
static size_t rows_i8_off(const QgLayout &L) { return gemm_workspace_least(L, QG_MAX_GROUPED); }
size_t qg_gemm_workspace_bytes(const QgLayout &L, int M)
{
    return M > 1 && qg_rows_i8_takes(L) ? rows_i8_off(L) + qg_rows_i8_bytes(L, M) : gemm_workspace_least(L, M);
}

extern "C" int qg_set_gemm_tuning(int splits, int shape)
{
    if (splits < 0 || splits > MAX_SPLITS || shape < -1 || shape > NSHAPES + 1) return QG_ERR_SHAPE;
    g_tune_splits = splits;
    g_tune_shape = shape;
    return QG_OK;
}

namespace {
// What one candidate of the launch-shape search costs, by the machine's budget (filled by a
// planning pass of gemm_small, which then enqueues nothing).
struct GemmPrice {
    int family;                // 0 raw codes, 1 gemm_rows16, 2 one GEMV per row, 3 dequantizing kernels
    int shape, splits;         // what the planner settled on (shape: index into SHAPES for family 3)
    long workgroups;           // of the main launch
    long iterations;           // barrier-to-barrier iterations one workgroup runs one after the other
    int launches;              // kernels the call enqueues
    KernelInfo kernel;
    double us;                 // family 0: what the plan says its kernels take
};

// The built-in plan of the dequantizing kernels: shape (index into SHAPES), workgroups along N and M, K ranges.
//   Up to 32 rows: one block of rows, two tiles x four
// k-slices.  Up to 64 rows: gemm_wide_b4 with four tiles per workgroup.  More: all rows
// in one wavefront (gemm_wide_b4, every weight dequantized once) when the launch has
// enough tiles for it, otherwise blocks of 64 rows on the grid's z axis, four tiles x two
// k-slices (two blocks double the wavefronts of a launch at the price of dequantizing
// twice, which pays as long as the launch cannot fill the chip).
struct DequantizingPlan {
    int shape, kw, tn, zblocks, blocks_x, steps_per_group, sps, splits;
};
DequantizingPlan dequantizing_plan(const QgLayout &L, int M, int cus, int knob_splits, int knob_shape)
{
    DequantizingPlan P;
    P.shape = M <= 32 ? 1 : M <= 64 ? 7 : L.tiles >= 128 ? 9 : 5;
    if (knob_shape > 0 && knob_shape <= NSHAPES) {
        const Shape &sh = SHAPES[knob_shape - 1];
        if (sh.wide ? (M > 32 && M <= sh.mb * 32) : ((sh.mb == 1) == (M <= 32))) P.shape = knob_shape - 1;
    }
    const int rows_per_block = SHAPES[P.shape].mb * 32;
    P.zblocks = (M + rows_per_block - 1) / rows_per_block;
    P.kw = SHAPES[P.shape].kw, P.tn = SHAPES[P.shape].tn;
    P.blocks_x = (int)((L.tiles + P.tn - 1) / P.tn);
    P.steps_per_group = L.group > KC ? L.group / KC : 1;
    // a split is a whole number of workgroup iterations and of groups
    const int quantum = P.kw / gcd(P.kw, P.steps_per_group) * P.steps_per_group;
    const int quanta = (int)((L.steps + quantum - 1) / quantum);
    // about one workgroup per compute unit, each with at least one quantum of work
    int splits = knob_splits ? knob_splits : (cus + P.blocks_x * P.zblocks - 1) / (P.blocks_x * P.zblocks);
    if (splits > MAX_SPLITS) splits = MAX_SPLITS;
    if (splits > quanta) splits = quanta;
    P.sps = (quanta + splits - 1) / splits * quantum;
    P.splits = (int)((L.steps + P.sps - 1) / P.sps);
    return P;
}
// What that plan costs: straight lines through 790 products of 28 matrices from 512 x 512 to 22016 x 8192, 17 ... 128 rows
// (root mean square of what they are off: 12 % up to 32 rows, 9 up to 64, 5 and 14 beyond).
double dequantizing_us(const QgLayout &L, int M, int cus)
{
    const DequantizingPlan P = dequantizing_plan(L, M, cus, 0, 0);
    struct Line { double call, round, iteration, iteration_full, g32, add, add_mb, y_mb; };
    static constexpr Line LINES[] = {{3.6, 0.0, 1.99, 0.06, 0.18, 2.3, 0.62, 0.0}, {3.6, 0.0, 2.3, 0.93, 0.05, 2.3, 0.23, 1.25},
                                     {3.6, 1.4, 2.57, 0.02, 0.11, 2.6, 0.14, 1.8}, {0.0, 0.0, 2.7, 2.5, 0.47, 7.5, 0.17, 1.24}};
    const Line &l = LINES[P.shape == 1 ? 0 : P.shape == 7 ? 1 : P.shape == 5 ? 2 : 3];
    const bool wide = SHAPES[P.shape].wide;
    const int most = P.sps < L.steps ? P.sps : (int)L.steps, iterations = (most + (wide ? 2 : P.kw) - 1) / (wide ? 2 : P.kw);
    const int64_t workgroups = (int64_t)P.blocks_x * P.zblocks * P.splits;
    const int capacity = cus * (wide ? 2 : 1);
    const int rounds = (int)((workgroups + capacity - 1) / capacity);
    const double full = workgroups < cus ? (double)workgroups / cus : 1.0, y_mb = 4e-6 * M * (double)L.N;
    double us = l.call + (rounds - 1) * l.round + l.y_mb * y_mb;
    us += rounds * iterations * (l.iteration + l.iteration_full * full + (L.group <= 32 ? l.g32 : 0.0));
    if (P.splits > 1) us += l.add + l.add_mb * P.splits * y_mb;
    return call_us(us, P.splits > 1 ? 2 : 1);
}

// What the product costs as M matrix-vector products in one launch (qg_gemv_rows): teams of eight wavefronts go through
// K, or the chip through all of the work.  Through 600 products of 2 ... 16 rows (9 % off below 11 us).
double gemv_rows_us(const QgLayout &L, int M)
{
    const double spw = (double)((L.steps + 7) / 8), step = (double)L.unit * L.step_units;
    const double per_step = L.group < step ? step / L.group : 1.0;
    const double work = 64e-9 * L.tiles * M * L.steps * step;
    const double one = ((L.bits == 4 ? 0.61 : 1.03) + 0.07 * per_step) * spw;
    const double all = ((L.bits == 4 ? 70.0 : L.bits == 3 ? 53.5 : 45.4) + 2.3 * per_step) * work;
    return 2.3 + sqrt(one * one + all * all);
}
// ... and on gemm_rows16: a workgroup per tile (teams of eight wavefronts, of four beyond one tile per compute unit).
// Through 4600 products of 2 ... 16 rows and 48 and more tiles, groups of 32 and more, two and more steps per wavefront (root mean square of what
// it is off: 7 %; 19 % at one step, where the caller is the longer).
double rows16_us(const QgLayout &L, int M, int cus)
{
    const int team = L.tiles > cus ? 4 : 8;
    const double rounds = (double)((L.tiles * team / 8 + cus - 1) / cus), spw = (double)((L.steps + team - 1) / team);
    const double full = L.tiles < cus ? (double)L.tiles / cus : 1.0;
    const double groups = L.group >= 128 ? 0.0 : L.group == 64 ? 0.27 : L.group == 32 ? 0.53 : 1.6;
    return 3.3 + rounds * spw * (0.73 + 0.023 * M + groups + 0.36 * full);
}

// Checks, plans and (price == NULL) enqueues one product; knob_*: as qg_set_gemm_tuning.
int gemm_small(const void *packed, int64_t N, int64_t K, int bits, int group, const float *X, int M,
               float *Y, void *workspace, size_t workspace_bytes, void *stream, int knob_splits,
               int knob_shape, GemmPrice *price)
{
    QgLayout L;
    const int rc = qg_make_layout(N, K, bits, group, &L);
    if (rc != QG_OK) return rc;
    if (M <= 0 || M > 128) return QG_ERR_SHAPE;
    if (!packed || !X || !Y) return QG_ERR_NULL;
    if (!qg_aligned16(packed) || ((uintptr_t)X & 63u) || !qg_aligned16(Y)) return QG_ERR_ALIGN;
    if (!workspace || workspace_bytes < gemm_workspace_least(L, M)) return QG_ERR_WORKSPACE;
    if (!qg_aligned16(workspace)) return QG_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;

    // One row of a 4-bit layout whose products of more rows leave parts of sums in the workspace (one row of the others is a
    // GEMV below): qg_gemv's arithmetic, in one launch that cuts no K over workgroups or, where a K is long for one, in a cut
    // launch, whose meeting slots a fill of 2 us empties first.  (As a bf16 product X was rounded, 1.7e-3 off 64
    // bits, now 1e-7; us per call 11008 x 4096 8.9 -> 6.7, 512 x 512 4.8 -> 2.6, 512 x 22016, cut, 17.2 -> 8.1.)
    const int gps = codes_gps(L);
    if (M == 1 && knob_shape == 0 && bits == 4 && (fast_path(L) || gps >= 0)) {
        if (call_us(gemv_rows_us(L, 1), 1) <= call_us(5.3 + 55e-9 * 64 * L.tiles * L.K, 2)) {
            const int r = qg_gemv_rows(packed, N, K, bits, group, X, 1, Y, stream, price != nullptr);
            if (r == QG_OK && price) *price = {2, -1, 1, 0, 0, 1, {nullptr, 0, 0}, 0.0};
            if (r != QG_ERR_UNSUPPORTED) return r;
        }
        const size_t slots = qg_workspace_bytes(N, K, bits, group, 1);
        const qg_gemv_desc d = {packed, N, K, bits, group, X, Y};
        int r = qg_gemv_grouped_check(&d, 1, workspace, slots);
        if (r == QG_OK && price) *price = {2, -1, 1, 0, 0, 2, {nullptr, 0, 0}, 0.0};
        if (r != QG_OK || price) return r;
        r = qg_workspace_init(workspace, slots, stream);
        return r == QG_OK ? qg_gemv_grouped_rows(&d, 1, workspace, slots, stream) : r;
    }

    // The raw-code kernel: every layout it takes that the 4-bit kernels below do not (2 and 3 bits, 4-bit
    // groups of 16), whatever shape 13 sends it, and the larger 4-bit matrices (in tile-steps of 64 outputs x
    // 128 k), where it is ahead of the dequantizing kernels; us per call, raw codes | dequantizing:
    //                            M = 24, g128, g32             M = 40, g128, g32
    //   5120 x 5120    (3200)  12.6 | 12.2  13.8 | 12.8      16.8 | 15.2  19.2 | 15.4
    //   4096 x 11008   (5504)  14.3 | 15.3  16.2 | 16.0      19.8 | 22.4  24.4 | 23.4
    //   11008 x 4096   (5504)  14.0 | 17.2  16.0 | 17.9      19.4 | 18.7  21.9 | 18.9
    //   8192 x 8192    (8192)  15.7 | 17.8  18.0 | 18.8      20.7 | 21.2  23.6 | 22.4
    //   13824 x 5120   (8640)  16.4 | 22.8  18.7 | 23.7      20.6 | 29.9  24.7 | 30.5
    //   5120 x 13824   (8640)  17.4 | 24.7  19.8 | 25.9      21.6 | 26.3  27.4 | 27.6
    // so at 33 ... 64 rows the line lies higher, and above 8192 for groups of 32, whose fold is as much work as their matrix
    // instructions.
    // Whatever else of more than 16 rows the dequantizing kernels take goes to the raw-code kernel where its price is the lower
    // one by more than the two are off.  That is most of all where groups are long: the dequantizing kernels cut K between
    // groups only (1500 x 20480, one group per output, M = 33 196 -> 19 us; 8192 x 8192 M = 8 37 -> 15), and 33 and more rows
    // of few tiles (1024 x 8192 g128 M = 96 17.6 -> 14.9, 4096 x 4096 M = 128 18.9 -> 15.6).
    // Up to 16 rows the cheapest of three is taken: the raw-code kernel; at 4 bits gemm_rows16; and, up to about 60 M
    // weights times rows, one fp32 matrix-vector product per row, in one launch that takes no more of the caller's time than
    // one product does.  (500 products of 2 ... 16 rows: 0.80 of the kernels' time of the raw-code kernel and gemm_rows16 from
    // 128 tiles on; 2045 x 576 4-bit M = 3 7.0 | 3.4 us, 1062 x 640 2-bit M = 5 6.1 | 3.3.  The dequantizing kernels were
    // the fastest of none.)
    const int from = M > 32 && M <= 64 ? (gps >= 4 ? 8448 : 8192) : 4096;
    const bool large = M > 16 && L.tiles * L.steps >= from;
    bool raw = gps >= 0 && M > 1 && (knob_shape == NSHAPES + 1 || knob_shape == 0);
    bool rows16 = false;
    const int cus = qg_compute_units();
    double us16 = 1e30, us1 = 1e30;                       // of the other two families up to 16 rows
    if (raw && knob_shape == 0 && M <= 16) {
        if (fast_path(L) && L.group <= KC && L.tiles >= 48) us16 = call_us(rows16_us(L, M, cus), 1);
        us1 = call_us(1.05 * gemv_rows_us(L, M), 1, M);
    }
    CodesPlan C;
    C.us = call_us(CODES_LEAST_US, 1);
    bool planned = raw && us1 >= C.us;                    // (else rows of products are the cheaper whatever the plan)
    if (planned) C = codes_plan(L, gps, M, knob_splits, knob_shape != 0);
    if (raw && knob_shape == 0) {
        // (by the built-in counts of K ranges, also where one is forced)
        const double us = knob_splits && planned ? codes_plan(L, gps, M, 0, false).us : C.us;
        if (M > 16) {
            raw = !fast_path(L) || large || us * 1.08 < dequantizing_us(L, M, cus);
        } else {
            rows16 = us16 < us && us16 <= us1;
            if (us1 < us && us1 < us16) {
                const int r = qg_gemv_rows(packed, N, K, bits, group, X, M, Y, stream, price != nullptr);
                if (r == QG_OK && price) *price = {2, -1, 1, 0, 0, 1, {nullptr, 0, 0}, 0.0};
                if (r != QG_ERR_UNSUPPORTED) return r;
            }
            raw = !rows16;
        }
        if (raw && !planned) C = codes_plan(L, gps, M, knob_splits, false);
    }
    if (raw) {
        const CodesSpace W = codes_space(L, gps, M);
        char *ws = (char *)workspace;
        QgPrepArgs P;
        P.X = X;
        P.Xop = ws;
        P.M = M;
        P.K = (int)K;
        P.steps_padded = W.steps_padded;
        P.groupk = W.groupk;
        P.arrived = (uint32_t *)(ws + W.arrived_off);
        P.counters = C.fused ? (int)L.tiles * C.zblocks : 0;
        QgCodesArgs A;
        const char *base = (const char *)packed;
        A.codes = base + L.codes_off;
        A.scales = base + L.scales_off;
        A.zeros = base + L.zeros_off;
        A.tile_codes = (uint32_t)(L.units * L.planes * QG_WAVE * 16);
        A.tile_scales = (uint32_t)(L.ngroups * QG_WAVE * 4);
        A.tile_zeros = (uint32_t)(L.zwords * QG_WAVE * 4);
        A.Xop = ws;
        A.Y = Y;
        A.partial = ws + W.partial_off;
        A.arrived = (uint32_t *)(ws + W.arrived_off);
        A.M = M;
        A.N = (int)N;
        A.tiles = (int)L.tiles;
        A.steps_padded = W.steps_padded;
        A.group_magic = gps == 0 ? (uint32_t)(((1ull << 32) + group / KC - 1) / (group / KC)) : 0;
        A.zshift = C.zblocks == 4 ? 2 : C.zblocks / 2;
        A.zblocks = C.zblocks;
        A.per_die = C.mb == 1 && C.zblocks > 1;      // (13824 x 5120 3-bit M = 37 22.6 -> 20.6 us, 4096 x 11008 4-bit M = 128 28.7 -> 26.2)
        A.units = C.units;
        A.ranges = C.ranges;
        A.quota = C.quota;
        A.total = C.blocks * C.units;
        A.fused = C.fused;
        A.self = C.self;
        A.X = X;
        A.K = (int)K;
        A.kw = C.kw;
        auto main_kernel = [&](KernelInfo *query) {
            return bits == 4 ? qg_codes_launch_b4(gps, C.mb, A, C.workgroups, st, query)
                 : bits == 2 ? qg_codes_launch_b2(gps, C.mb, A, C.workgroups, st, query)
                             : qg_codes_launch_b3(gps, C.mb, A, C.workgroups, st, query);
        };
        // (the instance is looked up before anything is enqueued: a layout without one is an error
        // that leaves nothing behind)
        KernelInfo info = {nullptr, 0, 0};
        const int have = main_kernel(&info);
        if (have != QG_OK) return have;
        if (price) {
            *price = {0, NSHAPES + (M > 32 && C.mb == 1) + 2 * C.self, C.ranges, (long)C.workgroups, C.quota, C.kernels, info, C.kernels_us};
            return QG_OK;
        }
        if (!C.self) {
            if (bits == 4) qg_codes_prepare_b4(P, W.rows_padded, st);
            else if (bits == 2) qg_codes_prepare_b2(P, W.rows_padded, st);
            else qg_codes_prepare_b3(P, W.rows_padded, st);
            if (qg_launch_status() != QG_OK) return QG_ERR_DEVICE;
        }
        const int r = main_kernel(nullptr);
        if (r != QG_OK) return r;
        if (qg_launch_status() != QG_OK) return QG_ERR_DEVICE;
        if (C.parts > 1 && !C.fused) {
            const int64_t quads = L.tiles * ((M + 7) / 8) * 2;
            const int waves = quads * 4 <= 4096 ? 4 : 2;                 // per quad: up to about 16 wavefronts per compute unit
            hipLaunchKernelGGL(waves == 4 ? add_parts<1> : add_parts<2>, dim3((unsigned)(quads * waves)), dim3(64), 0, st, A.partial,
                               (int)L.tiles, (int)N, M, C.tn, 32 * C.mb, C.zblocks, C.units, C.ranges, C.quota, Y);
        }
        return qg_launch_status();
    }

    // Up to 16 rows: the barrier-free kernel on the GEMV's launch structure, where it applies.
    // It has one workgroup per tile and no split of K over workgroups, so it needs enough tiles
    // to cover the chip (shape -1 forces it).
    if (M <= 16 && (rows16 || knob_shape < 0)) {
        const int r = qg_gemm_rows16(packed, N, K, bits, group, X, M, Y, workspace, stream, price != nullptr);
        if (r == QG_OK && price) *price = {1, -1, 1, (long)L.tiles, 0, 1, {nullptr, 0, 0}, 0.0};
        if (r != QG_ERR_UNSUPPORTED) return r;
    }

    // 3-bit groups of 32 weights: fp32 all the way, as qg_gemv computes it (X to 2^-30 of the largest of 128 values), the
    // cheapest of three: the product on int8 matrix instructions, two or three launches; a matrix-vector product per row, 16
    // rows to a launch, with K cut over workgroups (below; 150 products of 2 ... 16 rows, 9 % off) or not.
    // (A workspace that holds the slots of the call's rows but not the int8 operands keeps the products per row.  Several
    // launches of rows take more of the caller's time for each row, and cut ones are planned twice: over 48 products of
    // 17 ... 40 rows the choice takes 1.01 of the best one's time, always the int8 kernel 1.10: int8 | rows 254 x 1696 M = 18
    // 17.7 | 7.9 us, 964 x 1344 M = 32 15.8 | 8.6.)
    if (M > 1 && qg_rows_i8_takes(L) && workspace_bytes >= qg_gemm_workspace_bytes(L, M)) {
        const int splits = qg_rows_i8_splits(L, M), full = M / QG_MAX_GROUPED, rest = M % QG_MAX_GROUPED, calls = full + (rest > 0);
        const double us8 = call_us(qg_rows_i8_us(L, M), splits > 1 ? 3 : 2);
        const double rows_us = (full > 0 ? full * gemv_rows_us(L, QG_MAX_GROUPED) : 0.0) + (rest > 0 ? gemv_rows_us(L, rest) : 0.0);
        const double us1 = call_us(1.05 * rows_us, calls, calls > 1 ? 2 * M : M);
        const double cut = call_us(calls * (3.55 + 1.3e-4 * L.K) + 65e-9 * 64 * L.tiles * M * L.K, calls, calls > 1 ? 6 * M : 3 * M);
        if (us1 < us8 && us1 <= cut) {
            // (the first pass only plans, so that an error leaves nothing enqueued)
            int r = QG_OK;
            for (int pass = price || calls > 1 ? 0 : 1; pass < (price ? 1 : 2) && r == QG_OK; ++pass)
                for (int m0 = 0; m0 < M && r == QG_OK; m0 += QG_MAX_GROUPED)
                    r = qg_gemv_rows(packed, N, K, bits, group, X + (size_t)m0 * K, M - m0 < QG_MAX_GROUPED ? M - m0 : QG_MAX_GROUPED,
                                     Y + (size_t)m0 * N, stream, pass == 0);
            if (r == QG_OK && price) *price = {2, -1, 1, 0, 0, calls, {nullptr, 0, 0}, 0.0};
            if (r != QG_ERR_UNSUPPORTED) return r;
        }
        if (us8 <= cut) {
            if (price) {
                *price = {2, -1, splits, 0, 0, splits > 1 ? 3 : 2, {nullptr, 0, 0}, 0.0};
                return QG_OK;
            }
            float *partial = nullptr;
            const int r = qg_rows_i8(packed, L, X, M, Y, (char *)workspace + rows_i8_off(L), st, &partial);
            if (r != QG_OK || splits == 1) return r;
            const size_t count = (size_t)M * N;
            hipLaunchKernelGGL(add_splits, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, (const float *)partial, splits, count, Y);
            return qg_launch_status();
        }
    }

    if (!fast_path(L)) {
        // the fp32 GEMV once per activation row, up to 16 rows per launch (rows of X stay
        // 64-byte aligned only if K % 16 == 0)
        if (K % 16 != 0 && M > 1) return QG_ERR_UNSUPPORTED;
        // two passes over the launches of 16 rows: the first only checks and plans, so that an
        // error leaves nothing enqueued (a single launch sees to that itself)
        for (int pass = price || M > QG_MAX_GROUPED ? 0 : 1; pass < (price ? 1 : 2); ++pass)
            for (int m0 = 0; m0 < M; m0 += QG_MAX_GROUPED) {
                qg_gemv_desc d[QG_MAX_GROUPED];
                const int rows = M - m0 < QG_MAX_GROUPED ? M - m0 : QG_MAX_GROUPED;
                for (int i = 0; i < rows; ++i) {
                    d[i].packed = packed;
                    d[i].N = N;
                    d[i].K = K;
                    d[i].bits = bits;
                    d[i].group = group;
                    d[i].x = X + (size_t)(m0 + i) * K;
                    d[i].y = Y + (size_t)(m0 + i) * N;
                }
                const int r = pass == 0 ? qg_gemv_grouped_check(d, rows, workspace, workspace_bytes)
                                        : qg_gemv_grouped_rows(d, rows, workspace, workspace_bytes, stream);
                if (r != QG_OK) return r;
            }
        if (price) *price = {2, -1, 1, 0, 0, (M + QG_MAX_GROUPED - 1) / QG_MAX_GROUPED, {nullptr, 0, 0}, 0.0};
        return QG_OK;
    }

    const DequantizingPlan D = dequantizing_plan(L, M, qg_compute_units(), knob_splits, knob_shape);
    const int splits = D.splits;

    GemmArgs A;
    const char *base = (const char *)packed;
    A.codes = (const uint4 *)(base + L.codes_off);
    A.scales = (const float *)(base + L.scales_off);
    A.zeros = (const uint32_t *)(base + L.zeros_off);
    float *partial = (float *)workspace;
    A.X = X;
    A.out = splits > 1 ? partial : Y;
    A.M = M;
    A.N = (int)N;
    A.K = (int)K;
    A.tiles = (int)L.tiles;
    A.steps = (int)L.steps;
    A.ngroups = (int)L.ngroups;
    A.zwords = (int)L.zwords;
    A.group_shift = group == 32 ? 5 : group == 64 ? 6 : 7;
    A.steps_per_group = D.steps_per_group;
    A.steps_per_split = D.sps;
    const dim3 grid((unsigned)D.blocks_x, (unsigned)splits, (unsigned)D.zblocks);
    if (price) {
        KernelInfo info = {nullptr, 0, 0};
        launch_shape(D.shape, A, grid, st, &info);
        // (gemm_wide_b4 runs two steps per iteration)
        *price = {3, D.shape, splits, (long)D.blocks_x * splits * D.zblocks, D.sps / (SHAPES[D.shape].wide ? 2 : D.kw) + 1,
                  splits > 1 ? 2 : 1, info, 0.0};
        return QG_OK;
    }
    launch_shape(D.shape, A, grid, st);
    if (qg_launch_status() != QG_OK) return QG_ERR_DEVICE;
    if (splits > 1) {
        const size_t count = (size_t)M * N;
        hipLaunchKernelGGL(add_splits, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                           (const float *)partial, splits, count, Y);
    }
    return qg_launch_status();
}
}  // namespace

void qg_gemm_clear_tuning()
{
    std::lock_guard<std::mutex> lock(g_gemm_mutex);
    g_gemm_count = 0;
    g_gemm_next = 0;
}

extern "C" int qg_gemm_small(const void *packed, int64_t N, int64_t K, int bits, int group,
                             const float *X, int M, float *Y, void *workspace,
                             size_t workspace_bytes, void *stream)
{
    int splits = g_tune_splits, shape = g_tune_shape;
    if (splits == 0 && shape == 0 && g_gemm_count > 0) (void)gemm_tuning_for(N, K, bits, group, M, &splits, &shape);
    return gemm_small(packed, N, K, bits, group, X, M, Y, workspace, workspace_bytes, stream, splits, shape, nullptr);
}

// The launch-shape search of the small-M product: the counterpart of the paper's parameter search
// (Section 3, Algorithm 4, with the resource model of eqs. (3)-(5)) for this call.  Candidates
// are (kernel family / workgroup shape) x (number of K ranges).  Each is planned without being
// launched (a shape that does not fit the problem falls back to the built-in one, and a plan
// seen before is not tried again) and priced by its kernels: a raw-code cut by the built-in plan's estimate of
// them without the caller's time, the dequantizing kernels by the registers per lane and the LDS per workgroup
// of the instance, which give the workgroups the chip holds at once, hence the rounds the launch needs; a round
// costs a workgroup's fixed time plus its iterations, and every further kernel of the call a launch.
// Candidates priced above 1.5 times the cheapest are dropped, except the plan of the built-in choice, so that
// the search never records a slower one; the others are timed.
namespace {
constexpr int GT_SHAPES = NSHAPES + 3;           // 0 (built-in choice), -1 (gemm_rows16), 1 ... NSHAPES, NSHAPES + 1 (raw codes)
constexpr int GT_CANDIDATES = GT_SHAPES * MAX_SPLITS;
constexpr int gt_shape(int c) { return c / MAX_SPLITS == 0 ? 0 : c / MAX_SPLITS == 1 ? -1 : c / MAX_SPLITS - 1; }
float g_gt_us[GT_CANDIDATES];                    // -1: dropped by the price, -2: same plan as an earlier candidate
int g_gt_timed = 0, g_gt_dropped = 0;
// the dequantizing kernels, measured on this machine: a workgroup's time outside its loop (first loads, reduction across
// k-slices, output), one barrier-to-barrier iteration (a memory round trip), one more kernel in a call (the
// raw-code kernel has a unit's time by rows and groups, codes_cost_us, half to one and a half of that iteration)
constexpr double GT_FIXED_US = 3.3, GT_ITERATION_US = 2.0, GT_LAUNCH_US = 3.0;

double gemm_price_us(const GemmPrice &p)
{
    if (p.family == 0) return p.us;
    if (p.family == 1 || p.family == 2) return 0.0;          // no model: always timed
    int resident = 1;
    hipFuncAttributes attr;
    if (p.kernel.kernel && hipFuncGetAttributes(&attr, p.kernel.kernel) == hipSuccess) {
        const int waves = p.kernel.threads / QG_WAVE;
        const int regs = ((attr.numRegs > 0 ? attr.numRegs : 128) + 7) / 8 * 8;
        int per_simd = 512 / regs;
        if (per_simd > 8) per_simd = 8;
        if (per_simd < 1) per_simd = 1;
        resident = per_simd * 4 / waves;
        const size_t lds = attr.sharedSizeBytes + p.kernel.lds_dynamic;
        if (lds > 0 && (int)((160u << 10) / lds) < resident) resident = (int)((160u << 10) / lds);
        if (resident < 1) resident = 1;
    } else {
        (void)hipGetLastError();
    }
    const long capacity = (long)resident * qg_compute_units();
    const long rounds = (p.workgroups + capacity - 1) / capacity;
    return (double)rounds * (GT_FIXED_US + (double)p.iterations * GT_ITERATION_US) + (double)(p.launches - 1) * GT_LAUNCH_US;
}
}  // namespace

extern "C" int qg_gemm_autotune(const void *const *packed_sets, int sets, int64_t N, int64_t K, int bits,
                                int group, const float *X, int M, float *Y, void *workspace,
                                size_t workspace_bytes, void *stream, int repeats, int *splits,
                                int *shape, float *best_us)
{
    if (repeats <= 0 || sets <= 0) return QG_ERR_SHAPE;
    if (!packed_sets) return QG_ERR_NULL;
    for (int s = 0; s < sets; ++s)
        if (!packed_sets[s]) return QG_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    // 1. plan and price every candidate
    GemmPrice plan[GT_CANDIDATES];
    double price[GT_CANDIDATES], cheapest = -1.0;
    bool valid[GT_CANDIDATES];
    GemmPrice own;                                       // of the built-in choice
    const bool have_own = gemm_small(packed_sets[0], N, K, bits, group, X, M, Y, workspace, workspace_bytes, stream, 0, 0, &own) == QG_OK;
    auto same_plan = [](const GemmPrice &a, const GemmPrice &b) { return a.family == b.family && a.shape == b.shape && a.splits == b.splits; };
    for (int c = 0; c < GT_CANDIDATES; ++c) {
        const int sh = gt_shape(c), sp = 1 + c % MAX_SPLITS;
        const int rc = gemm_small(packed_sets[0], N, K, bits, group, X, M, Y, workspace, workspace_bytes, stream, sp, sh, &plan[c]);
        if (rc == QG_ERR_UNSUPPORTED) { valid[c] = false; continue; }
        if (rc != QG_OK) return rc;
        valid[c] = true;
        for (int e = 0; e < c && valid[c]; ++e)          // a knob the planner did not follow: seen already
            if (valid[e] && same_plan(plan[e], plan[c])) valid[c] = false;
        if (!valid[c]) continue;
        price[c] = gemm_price_us(plan[c]);
        if (price[c] > 0.0 && (cheapest < 0.0 || price[c] < cheapest)) cheapest = price[c];
    }
    // 2. time the survivors
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return QG_ERR_DEVICE;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return QG_ERR_DEVICE; }
    int best = -1, rc = QG_OK, turn = 0;
    float best_ms = -1.0f;
    g_gt_timed = 0;
    g_gt_dropped = 0;
    for (int c = 0; c < GT_CANDIDATES && rc == QG_OK; ++c) {
        g_gt_us[c] = -2.0f;
        if (!valid[c]) continue;
        if (price[c] > 1.5 * cheapest && cheapest > 0.0 && !(have_own && same_plan(plan[c], own))) {
            g_gt_us[c] = -1.0f;
            ++g_gt_dropped;
            continue;
        }
        const int sh = gt_shape(c), sp = 1 + c % MAX_SPLITS;
        auto run = [&]() {
            return gemm_small(packed_sets[turn++ % sets], N, K, bits, group, X, M, Y, workspace, workspace_bytes, stream, sp, sh, nullptr);
        };
        for (int i = 0; i < 2 && rc == QG_OK; ++i) rc = run();
        if (rc != QG_OK) break;
        if (hipEventRecord(e0, st) != hipSuccess) { rc = QG_ERR_DEVICE; break; }
        for (int i = 0; i < repeats && rc == QG_OK; ++i) rc = run();
        if (hipEventRecord(e1, st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) rc = QG_ERR_DEVICE;
        float ms = 0.0f;
        if (rc == QG_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = QG_ERR_DEVICE;
        if (rc != QG_OK) break;
        g_gt_us[c] = ms * 1e3f / (float)repeats;
        ++g_gt_timed;
        if (best < 0 || ms < best_ms) {
            best_ms = ms;
            best = c;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != QG_OK || best < 0) return rc != QG_OK ? rc : QG_ERR_DEVICE;
    const int won_shape = gt_shape(best), won_splits = 1 + best % MAX_SPLITS;
    gemm_record_tuning(N, K, bits, group, M, won_splits, won_shape);
    if (splits) *splits = won_splits;
    if (shape) *shape = won_shape;
    if (best_us) *best_us = best_ms * 1e3f / (float)repeats;
    return QG_OK;
}

extern "C" int qg_gemm_autotune_report(float *us, int capacity, int *timed, int *dropped)
{
    if (us) {
        if (capacity < GT_CANDIDATES) return QG_ERR_SHAPE;
        for (int c = 0; c < GT_CANDIDATES; ++c) us[c] = g_gt_us[c];
    }
    if (timed) *timed = g_gt_timed;
    if (dropped) *dropped = g_gt_dropped;
    return QG_OK;
}
