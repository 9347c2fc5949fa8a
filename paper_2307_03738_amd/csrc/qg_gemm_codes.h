// The small-M product with the weights entering the matrix instruction as RAW CODES: kernels and
// their launch interface.  Included by one source per bit width (qg_gemm_codes_b{2,3,4}.hip), each of
// which instantiates its width; qg_gemm_small.hip plans and launches.
//
// Nothing is dequantized per weight.  A code q becomes the exact bf16 integer 128 + q with a mask
// and an OR, the matrix instruction accumulates
//     T[m][n] = sum_{k in group} xb[m][k] (128 + q[n][k]),      xb = X rounded to bf16,
// in fp32 (the products are exact), and scale and zero-point are applied once per group and
// accumulator element, which is eq. (2) per element of Y:
//     Y[m][n] += s[n][g] * ( T[m][n] - (128 + z[n][g]) * xhat[m][g] ),   xhat[m][g] = sum_k xb[m][k].
// The subtraction rides on the matrix cores as well: xhat, cut into three bf16 parts (exact), is one
// more A operand per group and -(128 + z) one more B operand, so a group costs one fused
// multiply-add per accumulator element and nothing else on the vector ALU.
// (2 and 3 bits: every second field stays where it is, one field up, so half of the codes enter as
// 128 + 4 q or 128 + 8 q against activations stored divided by as much; those have an xhat of their
// own and the offset 32 or 16.)
//
// prepare_x converts X once per call into the A operands themselves: for every block of 32 rows and
// every step of 128 k, SEQ operands of 1 KB -- per group its xhat operand, then its k in sixteens -- each
// laid out as the 64 lanes of a wavefront read it (row = lane % 32, k-octet = lane / 32).  Rows past M
// and k past K are zeros, so the product kernel tests neither.  Blocks of 32 rows can also make their operands
// themselves, from X into LDS (SELF): every block of outputs converts X again, but a kernel less is launched, which
// is 2 us of the caller's time and 2 to 3 us on the GPU, against 0.1 us per unit up to 16 rows and 0.6 beyond (a unit
// itself 1.1 to 1.6).  So it is taken wherever units per workgroup are few (codes_price): 400 random products of
// 2 ... 32 rows take 0.80 of the time, 400 of 33 ... 128 rows 0.90; 1192 x 11200 3-bit g64 M = 5 12.4 -> 10.4 us,
// 1087 x 768 4-bit g128 M = 4 9.0 -> 6.5, 1408 x 3840 2-bit M = 38 11.9 -> 9.6.
//
// gemm_codes: a wavefront owns a tile of 64 outputs (device layout, lane = output) and MB blocks of 32
// rows; one v_permlane32_swap per pair of code words turns "lane = output" into the operand layout.  A
// workgroup is TN tiles x KW k-slices of wavefronts that share the A operands of a unit (KW steps) in
// LDS.  The operands go there straight from memory (buffer_load ... lds: no registers, no stores, no
// bank conflicts, since an operand is read as it lies), and every load of unit u + 1 is issued between
// the matrix instructions of unit u.  The units of the blocks of outputs and rows are cut into whole ranges of K
// or, where those would leave compute units idle, dealt evenly over one workgroup per compute unit, wherever the
// borders fall (22016 x 8192 at 128 rows: 172 workgroups with whole ranges, 251 dealt); with more blocks than
// compute units a workgroup takes a block.  More than 32 rows go in blocks of 64 or of 32 (codes_plan says when); several
// blocks of 32 rows of the same tiles sit in one die's workgroups, so that its L2 serves their weights.
//
// What bounds it: the issue of a SIMD.  A matrix instruction takes 12 cycles of it (measured: n multiply-adds behind
// each make max(34, 12 + 4 n) cycles, whether one wavefront runs on the SIMD or two).  Per 16 k x 64 outputs x 64 rows
// there are 4 matrix instructions and, at groups of 32 k, 32 multiply-adds of the fold plus 16-20 instructions of
// unpacking (4 cycles each): 2350 cycles per step of 128 k, 2-bit g32, of 2800 measured.  On short problems the
// launches around it count as much: prepare_x and, where many parts of a sum are better, add_parts.
// Measured (us per call, passes in sequence, four rotated matrices; before: iterations of KW layout steps,
// activations through registers, whole K ranges per block, always a kernel that adds the ranges): 22016 x
// 8192 2-bit g32 M = 128 104.4 -> 76, 13824 x 5120 3-bit g64 M = 37 27.0 -> 22.1 (in blocks of 32 rows 20.0), 4096 x 11008
// 4-bit g128 M = 128 28.2 -> 24.9.  Figures further down are differences that one choice made at the time it was taken.
#pragma once

#include <atomic>
#include <type_traits>

#include "qg_common.h"
#include "qg_mma.h"

struct QgCodesArgs {
    const char *codes, *scales, *zeros;
    const char *Xop;           // A operands (prepare_x)
    float *Y;
    char *partial;             // partial results [segment][tile][band of 8 rows][outputs 0-31, 32-63][lane][4 rows]
    uint32_t *arrived;         // [tile][block of rows]: workgroups whose part of the sum is there (prepare_x clears it)
    int M, N, tiles;
    uint32_t tile_codes, tile_scales, tile_zeros;      // bytes of one tile's codes, scales, zero words
    int steps_padded;          // steps of 128 k rounded up to a multiple of 4: what prepare_x has written
    uint32_t group_magic;      // groups of several steps: 2^32 / steps per group, rounded up
    int zshift;                // log2 of zblocks, if that is no three
    int units;                 // units (KW steps) in K
    int ranges;                // > 0: every block's units are cut into this many ranges, one workgroup each
    int quota;                 // units per workgroup
    int total;                 // units of the launch = blocks * units
    int fused;                 // parts of a sum are added here (else by add_parts)
    int kw;                    // k-slices of a workgroup
    int zblocks;               // blocks of 32 * MB rows: 1 ... 4
    int per_die;               // the workgroups of a die take neighbouring units: row blocks of a tile share its weights in L2
    int self;                  // the A operands are made here, from X
    int K;
    const float *X;            // [M][K] fp32
};

struct QgPrepArgs {
    const float *X;            // [M][K] fp32
    char *Xop;
    int M, K, steps_padded;
    int groupk;                // k one xhat covers: the group, or a step for groups of several steps
    uint32_t *arrived;         // counters the product kernel finds at zero
    int counters;
};

// What a launch would run, for the search that prices candidates before it times them.
struct QgKernelInfo {
    const void *kernel;
    int threads;
    size_t lds_dynamic;
};

// Variants of the product kernel.
enum {
    QG_CODES_PREPARED = 0,     // A operands by prepare_x, parts by add_parts
    QG_CODES_FUSED = 1,        // A operands by prepare_x, parts by the workgroup that comes last
    QG_CODES_SELF = 2          // A operands by the product kernel itself (blocks of 32 rows), parts by add_parts
};

constexpr size_t QG_LDS_BYTES = 160u << 10;
constexpr int QG_MAX_SEGMENTS = 8;             // parts the sum of an element of Y is cut into, at most
constexpr int QG_FUSED_SEGMENTS = 3;           // ... and are added by the workgroup that comes last, at most

// gps: groups per step of 128 k, 0 for groups of several steps.  A operands per step and block of 32 rows:
constexpr int qg_codes_seq(int gps) { return 8 + (gps > 0 ? gps : 1); }
// LDS of an instance: two units of A operands, and 32 rows of the accumulators of k-slices 1 ... KW-1; where
// those do not fit beside the operands (groups of 16 with four slices) they lie over the unit just multiplied
constexpr size_t qg_codes_stages(int gps, int mb, int kw) { return (size_t)2 * mb * kw * qg_codes_seq(gps) * 1024; }
constexpr bool qg_codes_slices_apart(int gps, int mb, int tn, int kw)
{
    return qg_codes_stages(gps, mb, kw) + (size_t)(kw - 1) * tn * 32 * 256 <= QG_LDS_BYTES;
}
constexpr size_t qg_codes_lds(int gps, int mb, int tn, int kw)
{
    return qg_codes_stages(gps, mb, kw) + (qg_codes_slices_apart(gps, mb, tn, kw) ? (size_t)(kw - 1) * tn * 32 * 256 : 0);
}
// k-slices of a workgroup of eight wavefronts: 4 at 32 rows and 2 at 64 (4 there, with half of the tiles, halves
// the partial sums but doubles the A operands' traffic: 13824 x 5120 3-bit M = 37 +3.0 us, 4096 x
// 11008 4-bit M = 128 +1.8; 1 doubles the partial sums: +0.3, +3.7; 2 at 32 rows: 4096 x 4096 +0.4, 4096 x 11008 +1.5 to
// 2, but 8192 x 22016 -1 to -1.5).  Groups of 16 at 32
// rows, with two A operands for every 16 k, are bound by that traffic as soon as there are tiles enough for
// every compute unit: 2 there (22016 x 8192 M = 2 40.6 against 45.4 us, 8192 x 8192 18.7 against 20.2), 4 below
// (1500 x 20480 29.4 against 20.2, 4096 x 11008 21.1 against 17.9, 512 x 512 9.2 against 8.1).
constexpr int qg_codes_kw(int gps, int mb, bool many_tiles) { return mb == 1 && !(gps == 8 && many_tiles) ? 4 : 2; }

// One per bit width.  query: fill it instead of launching.
int qg_codes_launch_b2(int gps, int mb, const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query);
int qg_codes_launch_b3(int gps, int mb, const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query);
int qg_codes_launch_b4(int gps, int mb, const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query);
void qg_codes_prepare_b2(const QgPrepArgs &P, int rows_padded, hipStream_t st);
void qg_codes_prepare_b3(const QgPrepArgs &P, int rows_padded, hipStream_t st);
void qg_codes_prepare_b4(const QgPrepArgs &P, int rows_padded, hipStream_t st);

#ifdef QG_CODES_KERNELS
namespace {

// One item = OCT consecutive k of one row (a cell at 2 bits, a word of a cell otherwise).  A workgroup takes
// one step of 32 rows and so writes its A operands whole: with a workgroup per row every 128-byte line of
// them was put together from eight workgroups' 16-byte pieces on different dies (a call with 128
// rows: 1.3 us on 4096 x 11008 4-bit, 1.6 on 22016 x 8192 2-bit).  Consecutive threads take
// consecutive items of a row, so the items of one xhat sit in neighbouring lanes.
template <int BITS>
__global__ __launch_bounds__(32 * 128 / (BITS == 2 ? 16 : 8)) void prepare_x(const QgPrepArgs A)
{
    constexpr int OCT = BITS == 2 ? 16 : 8;
    constexpr int S = 128, ITEMS = S / OCT, THREADS = 32 * ITEMS;
    // codes that are taken where they stand, one field further up: they enter as 128 + 8 q (3 bits)
    // or 128 + 4 q (2 bits) against activations divided by as much
    constexpr float UP = BITS == 3 ? 8.0f : 4.0f;
    const int step = blockIdx.x, item = threadIdx.x % ITEMS;
    const int m = blockIdx.y * 32 + threadIdx.x / ITEMS;
    for (int i = (blockIdx.y * gridDim.x + blockIdx.x) * THREADS + threadIdx.x; i < A.counters; i += gridDim.x * gridDim.y * THREADS) A.arrived[i] = 0u;
    const int in_step = item * OCT, k0 = step * S + in_step;
    const bool real = m < A.M && k0 < A.K;
    float val[OCT];
    if (real) {
        const float4 *src = (const float4 *)(A.X + (size_t)m * A.K + k0);
#pragma unroll
        for (int q = 0; q < OCT / 4; ++q) {
            const float4 v = src[q];
            val[4 * q + 0] = v.x; val[4 * q + 1] = v.y; val[4 * q + 2] = v.z; val[4 * q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < OCT; ++e) val[e] = 0.0f;
    }
    uint16_t h[OCT];                    // bf16 patterns in operand order: [operand][element]
    float sum0 = 0.0f, sum1 = 0.0f;
#pragma unroll
    for (int e = 0; e < OCT; e += 2) {
        const bool up0 = BITS == 3 ? (e & 7) >= 4 : false;                        // code e
        const bool up1 = BITS == 3 ? up0 : BITS == 2;                             // code e + 1
        mma_floatx2 t2 = {val[e] * (up0 ? 1.0f / UP : 1.0f), val[e + 1] * (up1 ? 1.0f / UP : 1.0f)};
        const mma_bf16x2 hb = __builtin_convertvector(t2, mma_bf16x2);            // round to nearest even
        const uint32_t bits = *(const uint32_t *)&hb;
        h[mma_slot<BITS>(e)] = (uint16_t)bits;
        h[mma_slot<BITS>(e + 1)] = (uint16_t)(bits >> 16);
        if (up0) sum1 += __uint_as_float(bits << 16) * UP; else sum0 += __uint_as_float(bits << 16);
        if (up1) sum1 += __uint_as_float(bits & 0xffff0000u) * UP; else sum0 += __uint_as_float(bits & 0xffff0000u);
    }
    // operand numbers: per group of the step its xhat, then its sixteens of k
    const int gk = A.groupk / 16;                          // sixteens per xhat
    const int per_group = gk + 1, seq = S / A.groupk * per_group;
    char *base = A.Xop + ((size_t)(m >> 5) * A.steps_padded + step) * seq * 1024 + (m & 31) * 16;
#pragma unroll
    for (int o = 0; o < OCT / 8; ++o) {
        uint4 piece;
        piece.x = h[8 * o + 0] | ((uint32_t)h[8 * o + 1] << 16);
        piece.y = h[8 * o + 2] | ((uint32_t)h[8 * o + 3] << 16);
        piece.z = h[8 * o + 4] | ((uint32_t)h[8 * o + 5] << 16);
        piece.w = h[8 * o + 6] | ((uint32_t)h[8 * o + 7] << 16);
        // 2 bits: cells 2 c and 2 c + 1 are the halves of operands 2 c and 2 c + 1
        const int k16 = BITS == 2 ? (in_step >> 5) * 2 + o : in_step >> 4;
        const int half = BITS == 2 ? (in_step >> 4) & 1 : (in_step >> 3) & 1;
        const int at = k16 / gk * per_group + 1 + k16 % gk;
        *(uint4 *)(base + at * 1024 + half * 512) = piece;
    }
    // xhat: the groupk / OCT neighbouring lanes hold its items (every lane takes part)
    const int wr = A.groupk / OCT;
    for (int off = 1; off < wr; off *= 2) {
        sum0 += __shfl_xor(sum0, off, 64);
        sum1 += __shfl_xor(sum1, off, 64);
    }
    if (item % wr == 0) {
        uint32_t part[2][3];            // three bf16 parts that add up to the sum exactly
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float rest = c == 0 ? sum0 : sum1;
#pragma unroll
            for (int p3 = 0; p3 < 3; ++p3) {
                mma_floatx2 t2 = {rest, 0.0f};
                const mma_bf16x2 hb = __builtin_convertvector(t2, mma_bf16x2);
                part[c][p3] = *(const uint32_t *)&hb & 0xffffu;
                rest -= __uint_as_float(part[c][p3] << 16);
            }
        }
        char *ce = base + in_step / A.groupk * per_group * 1024;
        *(uint4 *)ce = make_uint4(part[0][0] | (part[0][1] << 16), part[0][2], 0u, 0u);
        *(uint4 *)(ce + 512) = make_uint4(part[1][0] | (part[1][1] << 16), part[1][2], 0u, 0u);
    }
}

typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ inline rsrc_t buffer_of(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000);
}

// HOW: QG_CODES_*.  FUSED: parts of a sum are added by the workgroup that comes last (an instance of its own: the code
// for it costs the others 3 %).
template <int BITS, int GPS_, int MB, int TN, int KW, int HOW>
__global__ __launch_bounds__(TN * KW * 64, 2) void gemm_codes(const QgCodesArgs A)
{
    using F = Fmt<BITS>;
    constexpr bool FUSED = HOW == QG_CODES_FUSED, SELF = HOW == QG_CODES_SELF;
    constexpr bool LONG = GPS_ == 0;                     // groups of several steps
    constexpr bool SHORT = GPS_ >= 2;                    // groups of 64 k or less: see compute_short
    constexpr int GPS = LONG ? 1 : GPS_;                 // xhat entries per step
    constexpr int NW = TN * KW;
    constexpr int L = BITS;                              // 128-bit code vectors per lane and step (128 k x 64 outputs)
    constexpr int GK = 8 / GPS;                          // sixteens of k per xhat
    constexpr int SEQ = GPS * (GK + 1);                  // A operands per step and row block
    constexpr int ROWS = 32 * MB;
    constexpr int CHUNK = MB * KW * SEQ;                 // KB of A operands per unit
    constexpr int NDMA = SELF ? 0 : (CHUNK + NW - 1) / NW;          // 1 KB copies per wavefront and unit
    constexpr int NLOAD = L + 1 + GPS;                   // weight loads per wavefront and unit
    constexpr int ZPER = 32 / F::ZBITS;
    constexpr int SLOTS = 2 * MB;                        // matrix instructions per A operand index
    static_assert(SEQ == qg_codes_seq(GPS_), "operand count");
    static_assert(NLOAD + NDMA <= SEQ * SLOTS, "a request per slot");
    static_assert(!SELF || (MB == 1 && NW >= 2 * KW), "a wavefront per 16 rows and step");
    extern __shared__ __attribute__((aligned(16))) char smem[];       // [2][CHUNK KB], then the reduction's

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tn = wave % TN, kw = wave / TN;
    const int half = lane >> 5, row = lane & 31;
    const uint32_t lane4 = lane * 4, lane16 = lane * 16;

    // this workgroup's units [u, u1) in the order (block of outputs, block of rows, unit of K)
    int wg = blockIdx.x;
    if (A.per_die) {                                     // workgroup i of the grid runs on die i % 8
        const int die = wg & 7, more = gridDim.x & 7;
        wg = die * (gridDim.x >> 3) + (die < more ? die : more) + (wg >> 3);
    }
    int u, u1, b;
    if (A.ranges > 0) {
        b = __builtin_amdgcn_readfirstlane(wg / A.ranges);
        u = b * A.units + (wg - b * A.ranges) * A.quota;
        u1 = u + A.quota;
        u1 = u1 < (b + 1) * A.units ? u1 : (b + 1) * A.units;
    } else {
        u = wg * A.quota;
        u1 = u + A.quota;
        u1 = u1 < A.total ? u1 : A.total;
        b = __builtin_amdgcn_readfirstlane(u / A.units);
    }
    int it = u - b * A.units;

    struct StepRegs {
        uint4 v[L];
        float s[GPS];
        uint32_t zw;
    };
    // Where the next unit's data are (all scalar).  Reads past a tile's codes, scales or zero words (a
    // k-slice past K; the last step of a K that ends inside it) return zeros; the activations there are
    // zeros too.  A buffer checks the lane's offset against its size and leaves the scalar offset of the
    // instruction out, so the buffers of a unit begin at its step and end with the tile's section (a step
    // past it: size 0).
    const char *codes_t, *scales_t, *zeros_t;
    rsrc_t codes_n, scales_n, zeros_n, x_n;
    uint32_t at_x;
    bool x_takes = false;                                // SELF: this wavefront converts a part of the unit's X
    const uint32_t x_row_block = (uint32_t)A.steps_padded * (SEQ * 1024);
    auto tiles_of = [&](int nb) { return A.zblocks == 3 ? (int)__umulhi((uint32_t)nb, 0x55555556u) : nb >> A.zshift; };
    auto aim_block = [&](int nb) {
        const int tb = tiles_of(nb), z = nb - tb * A.zblocks;
        int tile = tb * TN + tn;
        tile = tile < A.tiles ? tile : A.tiles - 1;
        codes_t = A.codes + (size_t)tile * A.tile_codes;
        scales_t = A.scales + (size_t)tile * A.tile_scales;
        zeros_t = A.zeros + (size_t)tile * A.tile_zeros;
        if constexpr (SELF) {
            const int rows = A.M - z * 32 < 32 ? A.M - z * 32 : 32;
            x_n = buffer_of(A.X + (size_t)z * 32 * A.K, (uint32_t)rows * A.K * 4);
            x_takes = wave < (rows > 16 ? 2 : 1) * KW;
        } else {
            x_n = buffer_of(A.Xop + (size_t)z * MB * x_row_block, MB * x_row_block);
        }
    };
    auto rest_of = [&](const char *section, uint32_t bytes, uint32_t at) {
        at = at < bytes ? at : bytes;
        return buffer_of(section + at, bytes - at);
    };
    auto aim = [&](int nit) {
        const uint32_t step = nit * KW + kw;
        const uint32_t g = LONG ? __umulhi(step, A.group_magic) : step * GPS;
        codes_n = rest_of(codes_t, A.tile_codes, step * (L * 1024));
        scales_n = rest_of(scales_t, A.tile_scales, g * 256);
        zeros_n = rest_of(zeros_t, A.tile_zeros, g / ZPER * 256);                         // a step's groups share one zero word
        at_x = SELF ? nit * (KW * 128) : nit * (KW * SEQ * 1024);
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    // pieces of a unit's A operands this wavefront copies: where they are in memory
    uint32_t piece_at[NDMA > 0 ? NDMA : 1];
#pragma unroll
    for (int j = 0; j < NDMA; ++j) {
        int p = j * NW + wave;
        p = p < CHUNK ? p : CHUNK - 1;                       // (the last piece again: same bytes to the same place)
        const int rb = p / (KW * SEQ);
        piece_at[j] = __builtin_amdgcn_readfirstlane(rb * x_row_block + (p - rb * (KW * SEQ)) * 1024);
    }
    // request t of a unit: codes, zero word, scales, then the wavefront's share of the A operands, which
    // go from memory to LDS without passing through registers
    auto request = [&](int t, StepRegs &r, int stage) {
        if (t < L) {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(codes_n, lane16 + t * 1024, 0, 0);
            r.v[t] = make_uint4(v[0], v[1], v[2], v[3]);
        } else if (t == L) {
            r.zw = __builtin_amdgcn_raw_buffer_load_b32(zeros_n, lane4, 0, 0);
        } else if (t < NLOAD) {
            r.s[t - L - 1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(scales_n, lane4 + (t - L - 1) * 256, 0, 0));
        } else if (t < NLOAD + NDMA) {
            const int j = t - NLOAD;
            const int p = j * NW + wave < CHUNK ? j * NW + wave : CHUNK - 1;
            const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + (stage * CHUNK + p) * 1024);
            const uint32_t from = __builtin_amdgcn_readfirstlane(at_x + piece_at[j]);
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"(lane16), "s"(x_n), "s"(from)
                         : "memory", "m0");
        }
    };

    // SELF.  A wavefront takes 16 rows of one step: lane 4 r + i loads items i (OCT consecutive k, as in prepare_x) of
    // row r of every quarter (2 bits: half) of the step, whole lines of X, while the unit before is multiplied, and
    // writes them as pieces of the A operands at the end of it.  Rows past M and k past K lie outside the buffer and
    // come as zeros.  The 16 bytes of row r of an operand's half lie at place r ^ 4 half ^ 8 parity of that half, parity
    // being bit 1 of the item: the four items and four rows that 16 lanes write then fall on distinct banks.
    constexpr int OCT = BITS == 2 ? 16 : 8, SUBS = 32 / OCT;          // (a lane's 32 values of a step)
    constexpr float UP = BITS == 3 ? 8.0f : 4.0f;
    const int x_item = lane & 3, x_row = (wave / KW & 1) * 16 + (lane >> 2);
    uint4 xr[SELF ? 8 : 1];
    bool x_loaded = false;
    auto load_x = [&]() {
        x_loaded = x_takes;
        if (!x_loaded) return;
        const uint32_t from = (uint32_t)x_row * A.K * 4;
#pragma unroll
        for (int s = 0; s < SUBS; ++s) {
            const uint32_t k = at_x + wave % KW * 128 + (4 * s + x_item) * OCT;
            const uint32_t at = k < (uint32_t)A.K ? from + k * 4 : 0x40000000u;      // (past every buffer of 32 rows)
#pragma unroll
            for (int i = 0; i < OCT / 4; ++i) {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(x_n, at + 16 * i, 0, 0);
                xr[s * (OCT / 4) + i] = make_uint4(v[0], v[1], v[2], v[3]);
            }
        }
    };
    auto quad_add = [](float v, auto ctrl) {
        return v + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    auto store_x = [&](int stage) {
        if (!x_loaded) return;
        const int xhalf = x_item & 1, par = x_item >> 1;
        char *to = smem + (stage * CHUNK + wave % KW * SEQ) * 1024 + xhalf * 512;
        const int place = (x_row ^ (4 * xhalf)) * 16;
        constexpr int PAIRS = SUBS * 4 * OCT / 16 / GK;               // xhats of the step
        static_assert(PAIRS == GPS, "xhats");
        float sum0 = 0.0f, sum1 = 0.0f;
#pragma unroll
        for (int s = 0; s < SUBS; ++s) {
            float t[OCT];                                             // in operand order
#pragma unroll
            for (int e = 0; e < OCT; ++e) {
                const bool up = BITS == 3 ? (e & 7) >= 4 : BITS == 2 && (e & 1);
                t[mma_slot<BITS>(e)] = __uint_as_float(word_of(xr[s * (OCT / 4) + e / 4], e & 3)) * (up ? 1.0f / UP : 1.0f);
            }
#pragma unroll
            for (int o = 0; o < OCT / 8; ++o) {
                MmaOperand piece;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const mma_floatx2 t2 = {t[8 * o + 2 * j], t[8 * o + 2 * j + 1]};
                    const mma_bf16x2 hb = __builtin_convertvector(t2, mma_bf16x2);      // round to nearest even
                    piece.r[j] = *(const uint32_t *)&hb;
                    // 2 and 3 bits: the registers of codes taken one field up
                    const bool up = BITS == 3 ? (j & 1) != 0 : BITS == 2 && (j & 1);
                    const float pair = __uint_as_float(piece.r[j] << 16) + __uint_as_float(piece.r[j] & 0xffff0000u);
                    if (up) sum1 += pair; else sum0 += pair;
                }
                // the lane's piece: sixteen c of the step, c = c0 at parity 0
                const int c0 = BITS == 2 ? 4 * s + o : 2 * s;
                const int next = BITS == 2 ? 2 : 1;                   // ... and c0 + next at parity 1
                const int at0 = c0 / GK * (GK + 1) + 1 + c0 % GK, at1 = (c0 + next) / GK * (GK + 1) + 1 + (c0 + next) % GK;
                *(lds_u128 *)(to + at0 * 1024 + par * ((at1 - at0) * 1024) + (place ^ (128 * par))) = piece.q;
            }
            constexpr int SUB16 = 4 * OCT / 16;                       // sixteens of k the four lanes hold
            if ((s + 1) * SUB16 % GK == 0) {
                // xhat of a group: over the four lanes, or over two of them where they hold two groups
                sum0 = quad_add(sum0, std::integral_constant<int, 0xb1>());
                sum1 = quad_add(sum1, std::integral_constant<int, 0xb1>());
                if constexpr (GK >= SUB16) {
                    sum0 = quad_add(sum0, std::integral_constant<int, 0x4e>());
                    sum1 = quad_add(sum1, std::integral_constant<int, 0x4e>());
                }
                float rest = xhalf ? (BITS == 4 ? 0.0f : sum1 * UP) : sum0;
                uint32_t part[3];
#pragma unroll
                for (int p3 = 0; p3 < 3; ++p3) {
                    const mma_floatx2 t2 = {rest, 0.0f};
                    const mma_bf16x2 hb = __builtin_convertvector(t2, mma_bf16x2);
                    part[p3] = *(const uint32_t *)&hb & 0xffffu;
                    rest -= __uint_as_float(part[p3] << 16);
                }
                const int grp = ((s + 1) * SUB16 - 1) / GK;           // GK < SUB16: of parity 1
                if (GK < SUB16) *(lds_u128 *)(to + ((grp - 1) + par) * ((GK + 1) * 1024) + place) = make_uint4(part[0] | (part[1] << 16), part[2], 0u, 0u);
                else if (par == 0) *(lds_u128 *)(to + grp * ((GK + 1) * 1024) + place) = make_uint4(part[0] | (part[1] << 16), part[2], 0u, 0u);
                sum0 = sum1 = 0.0f;
            }
        }
    };
    // where lane (row, half) finds its piece of an operand: the xhats and sixteens of parity 0, those of parity 1
    const uint32_t a_at0 = SELF ? half * 512 + (row ^ (4 * half)) * 16 : lane16, a_at1 = SELF ? a_at0 ^ 128 : lane16;
    auto a_at = [&](int q) {
        const int c = q / (GK + 1) * GK + q % (GK + 1) - 1;
        const bool odd = q % (GK + 1) != 0 && (BITS == 2 ? (c >> 1) & 1 : c & 1);
        return (odd ? a_at1 : a_at0) + q * 1024;
    };

    // ---- accumulators ----
    constexpr int NT = SHORT ? 2 : 2 * MB;
    mma_floatx16 acc[NT];                     // T of the running group: [2 mb + (outputs 0-31: 0, 32-63: 1)]; SHORT: of two tiles
    float y[2 * MB][16];
    const mma_floatx16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    float sP = 0.0f, sQ = 0.0f;               // scales of the group the accumulators belong to
    float sc[2][2];                           // SHORT: [outputs 0-31, 32-63][group parity]
    uint32_t held = ~0u;                      // LONG: that group
    auto reset = [&]() {
        // (an opaque zero: the accumulators must not be cleared ahead of the sums over parts, which want
        // their registers)
        float zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[k][i] = zero;
#pragma unroll
        for (int k = 0; k < 2 * MB; ++k)
#pragma unroll
            for (int i = 0; i < 16; ++i) y[k][i] = zero;
        sP = sQ = sc[0][0] = sc[0][1] = sc[1][0] = sc[1][1] = zero;
        held = ~0u;
    };
    auto fold = [&](int k) {
        const float s = (k & 1) ? sQ : sP;
#pragma unroll
        for (int i = 0; i < 16; ++i) y[k][i] = fmaf(s, acc[k][i], y[k][i]);
    };
    const MmaConst mc = mma_constants<BITS>();
    // bf16 -(128 + z); where codes are taken one field up, lanes 32-63: -(16 + z) (3 bits) or -(32 + z)
    // (2 bits) against the other xhat (4 bits: zeros meet it)
    const uint32_t corr_base = BITS == 3 && half ? 0xc180c180u : BITS == 2 && half ? 0xc200c200u : 0xc300c300u;
    const uint32_t corr_shift = BITS == 3 && half ? 3 : BITS == 2 && half ? 2 : 0;

    // One unit of this wavefront.  Matrix instruction k of operand index q is followed by a piece of the
    // preparation of index q + 1 (lane exchange, unpacking, LDS reads), by one request for the next unit
    // and, where a group starts, preceded by the fold of the group that ended.  Every slot is fenced, so
    // that the order written here is the order issued.
    auto compute = [&](const StepRegs &r, uint32_t step, int stage, StepRegs &req) {
        const char *xs = smem + (stage * CHUNK + kw * SEQ) * 1024;
        const uint32_t g = LONG ? __umulhi(step, A.group_magic) : step * GPS;             // first group of the step
        const uint32_t zw = r.zw >> (F::ZBITS * (g % ZPER));
        const auto zsw = __builtin_amdgcn_permlane32_swap(zw, zw, false, false);
        MmaOperand bP, bQ, nP, nQ, aC[MB], aN[MB];
        uint32_t wP = 0, wQ = 0;
        float nsP = 0.0f, nsQ = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) nP.r[j] = nQ.r[j] = 0u;
        auto swap = [&](uint32_t a, uint32_t c) {
            const auto sw = __builtin_amdgcn_permlane32_swap(a, c, false, false);
            wP = sw[0];           // outputs 0-31: a in lanes 0-31, c in lanes 32-63
            wQ = sw[1];           // outputs 32-63
        };
        // prepares operand index q in four parts
        auto part = [&](int q, int i) {
            const int grp = q / (GK + 1), rr = q % (GK + 1);
            if (rr == 0) {
                if (i == 0) {
                    const uint32_t m = (1u << F::ZBITS) - 1u;
                    const uint32_t zP = ((zsw[0] >> (F::ZBITS * grp)) & m) << corr_shift, zQ = ((zsw[1] >> (F::ZBITS * grp)) & m) << corr_shift;
                    nP.r[0] = nP.r[1] = corr_base | zP | (zP << 16);
                    nQ.r[0] = nQ.r[1] = corr_base | zQ | (zQ << 16);
                }
                if (i == 1 && !LONG) {
                    const auto ssw = __builtin_amdgcn_permlane32_swap(__float_as_uint(r.s[grp]), __float_as_uint(r.s[grp]), false, false);
                    nsP = __uint_as_float(ssw[0]);
                    nsQ = __uint_as_float(ssw[1]);
                }
                return;
            }
            const int c = grp * GK + rr - 1;                  // sixteen of k within the step
            if constexpr (BITS == 4) {
                if (i == 0) swap(word_of(r.v[c >> 1], 2 * (c & 1)), word_of(r.v[c >> 1], 2 * (c & 1) + 1));
            } else if constexpr (BITS == 2) {
                if (i == 0 && (c & 1) == 0) swap(word_of(r.v[c >> 2], c & 2), word_of(r.v[c >> 2], (c & 2) + 1));
            } else {
                const int cell = c >> 1;
                if (i == 0) {
                    const uint32_t wa = word_of(r.v[0], cell), wb = word_of(r.v[1], cell), wc = word_of(r.v[2], cell);
                    if ((c & 1) == 0) swap(wa, wb);
                    else swap(wc, ((wa >> 6) & 0x03030303u) | ((wb >> 4) & 0x0c0c0c0cu) | ((wc >> 2) & 0x30303030u));
                }
            }
            const uint32_t w = i < 2 ? wP : wQ;
            MmaOperand &o = i < 2 ? nP : nQ;
            const int j0 = 2 * (i & 1);
            if constexpr (BITS == 4) {
                o.r[j0] = and_or(w >> (4 * j0), mc.mask, mc.magic);
                o.r[j0 + 1] = and_or(w >> (4 * j0 + 4), mc.mask, mc.magic);
            } else {
                const uint32_t v = w >> (BITS == 3 ? 8 * (i & 1) : 2 * (j0 + 4 * (c & 1)));
                o.r[j0] = and_or(v, mc.mask, mc.magic);
                o.r[j0 + 1] = and_or(v, mc.mask_up, mc.magic);
            }
            asm volatile("" : "+v"(o.r[j0]), "+v"(o.r[j0 + 1]));      // keeps the piece in its slot
        };
        auto read_a = [&](int q, MmaOperand *a) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) a[mb].q = *(const lds_u128 *)(xs + mb * KW * SEQ * 1024 + a_at(q));
        };
        read_a(0, aN);
        if constexpr (LONG) {
            if (g != held) {                         // uniform: the running group ended before this step
#pragma unroll
                for (int k = 0; k < 2 * MB; ++k) {
                    fold(k);
                    acc[k] = zero16;
                }
                const auto ssw = __builtin_amdgcn_permlane32_swap(__float_as_uint(r.s[0]), __float_as_uint(r.s[0]), false, false);
                sP = __uint_as_float(ssw[0]);
                sQ = __uint_as_float(ssw[1]);
                held = g;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) part(0, i);
#pragma unroll
        for (int q = 0; q < SEQ; ++q) {
            const bool starts = !LONG && q % (GK + 1) == 0;
            const float tsP = nsP, tsQ = nsQ;
            bP = nP;
            bQ = nQ;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) aC[mb] = aN[mb];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < SLOTS; ++k) {
                if (starts) fold(k);
                acc[k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aC[k >> 1].v, (k & 1) ? bQ.v : bP.v, starts ? zero16 : acc[k], 0, 0, 0);
                if (q + 1 < SEQ) {
                    if (k == 0) read_a(q + 1, aN);
#pragma unroll
                    for (int i = 0; i < 4 / SLOTS; ++i) part(q + 1, k * (4 / SLOTS) + i);
                }
                request(q * SLOTS + k, req, stage ^ 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (starts) {
                sP = tsP;
                sQ = tsQ;
            }
        }
    };

    // The same for groups of 64 k and less, where the fold is as much work as the matrix instructions of a
    // group: in the order above all of a group's folds stand together and the matrix core waits for them.
    // Here a group is taken one tile of 32 rows x 32 outputs after the other, each a chain of GK + 1 matrix
    // instructions into one of two accumulators, and the fold of the tile before runs under the chain.
    // The operands of outputs 32-63 are prepared under the chains of outputs 0-31 and the other way round.
    auto compute_short = [&](const StepRegs &r, uint32_t step, int stage, StepRegs &req) {
        constexpr int R = GK + 1;                          // operands of a group: xhat, sixteens of k
        constexpr int PIECES = 2 * GK + 1;                 // pieces of preparation per half of a group
        const char *xs = smem + (stage * CHUNK + kw * SEQ) * 1024;
        const uint32_t zw = r.zw >> (F::ZBITS * (step * GPS % ZPER));
        const auto zsw = __builtin_amdgcn_permlane32_swap(zw, zw, false, false);
        MmaOperand bo[2][R], a[MB == 1 ? 2 : 1][MB][R];
        uint32_t w[2][GK];
#pragma unroll
        for (int j = 0; j < 4; ++j) bo[0][0].r[j] = bo[1][0].r[j] = 0u;
        // piece j of the operands of outputs 32 pq ... of group grp
        auto piece = [&](int pq, int grp, int j) {
            if (j == 0) {
                const uint32_t z = ((zsw[pq] >> (F::ZBITS * grp)) & ((1u << F::ZBITS) - 1u)) << corr_shift;
                bo[pq][0].r[0] = bo[pq][0].r[1] = corr_base | z | (z << 16);
                asm volatile("" : "+v"(bo[pq][0].r[0]), "+v"(bo[pq][0].r[1]));
                if (pq == 0) {
                    const auto ssw = __builtin_amdgcn_permlane32_swap(__float_as_uint(r.s[grp]), __float_as_uint(r.s[grp]), false, false);
                    sc[0][grp & 1] = __uint_as_float(ssw[0]);
                    sc[1][grp & 1] = __uint_as_float(ssw[1]);
                }
                return;
            }
            const int i = (j - 1) >> 1, h = (j - 1) & 1, c = grp * GK + i;      // operand, its half, sixteen of k within the step
            if (pq == 0 && h == 0 && (BITS != 2 || (c & 1) == 0)) {
                uint32_t x0, x1;
                if constexpr (BITS == 4) {
                    x0 = word_of(r.v[c >> 1], 2 * (c & 1));
                    x1 = word_of(r.v[c >> 1], 2 * (c & 1) + 1);
                } else if constexpr (BITS == 2) {
                    x0 = word_of(r.v[c >> 2], c & 2);
                    x1 = word_of(r.v[c >> 2], (c & 2) + 1);
                } else {
                    const uint32_t wa = word_of(r.v[0], c >> 1), wb = word_of(r.v[1], c >> 1), wc = word_of(r.v[2], c >> 1);
                    x0 = (c & 1) == 0 ? wa : wc;
                    x1 = (c & 1) == 0 ? wb : ((wa >> 6) & 0x03030303u) | ((wb >> 4) & 0x0c0c0c0cu) | ((wc >> 2) & 0x30303030u);
                }
                const auto sw = __builtin_amdgcn_permlane32_swap(x0, x1, false, false);
                w[0][i] = sw[0];
                w[1][i] = sw[1];
            }
            const uint32_t v = w[pq][BITS == 2 ? i & ~1 : i];
            MmaOperand &o = bo[pq][i + 1];
            if constexpr (BITS == 4) {
                o.r[2 * h] = and_or(v >> (8 * h), mc.mask, mc.magic);
                o.r[2 * h + 1] = and_or(v >> (8 * h + 4), mc.mask, mc.magic);
            } else {
                const uint32_t f = v >> (BITS == 3 ? 8 * h : 4 * h + 8 * (c & 1));
                o.r[2 * h] = and_or(f, mc.mask, mc.magic);
                o.r[2 * h + 1] = and_or(f, mc.mask_up, mc.magic);
            }
            asm volatile("" : "+v"(o.r[2 * h]), "+v"(o.r[2 * h + 1]));          // keeps the piece in its slot
        };
        auto read_a = [&](int grp, int mb) {
#pragma unroll
            for (int q = 0; q < R; ++q) a[MB == 1 ? grp & 1 : 0][mb][q].q = *(const lds_u128 *)(xs + mb * KW * SEQ * 1024 + a_at(grp * R + q));
        };
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) read_a(0, mb);
#pragma unroll
        for (int j = 0; j < PIECES; ++j) piece(0, 0, j);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int grp = 0; grp < GPS; ++grp)
#pragma unroll
            for (int t = 0; t < 2 * MB; ++t) {
                const int pq = t / MB, mb = t % MB;
                // the tile before this one, and its group's scale
                const int tp = t == 0 ? 2 * MB - 1 : t - 1;
                const float s = sc[tp / MB][(t == 0 ? grp + 1 : grp) & 1];
                float *yp = y[2 * (tp % MB) + tp / MB];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    acc[t & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[MB == 1 ? grp & 1 : 0][mb][q].v, bo[pq][q].v, q == 0 ? zero16 : acc[t & 1], 0, 0, 0);
                    if (q == 0) {
                        // rows whose operands nothing of this group needs any more, or (row block 1) needs next
                        if (MB == 1 && t == 0 && grp + 1 < GPS) read_a(grp + 1, 0);
                        if (MB == 2 && t == 3 && grp + 1 < GPS) read_a(grp + 1, 0);
                        if (MB == 2 && t == 0 && grp > 0) read_a(grp, 1);
                    }
                    // (behind the first instruction of a chain the tile before is not there yet: half of the
                    // chain's preparation goes there, the fold behind the others)
                    const int j0 = mb * PIECES / MB, jn = (mb + 1) * PIECES / MB - j0, jh = (jn + 1) / 2;
                    const int ja = q == 0 ? 0 : jh + (jn - jh) * (q - 1) / GK, jb = q == 0 ? jh : jh + (jn - jh) * q / GK;
#pragma unroll
                    for (int j = j0 + ja; j < j0 + jb; ++j) {
                        if (pq == 0) piece(1, grp, j);
                        else if (grp + 1 < GPS) piece(0, grp + 1, j);
                    }
                    if (q > 0) {
#pragma unroll
                        for (int i = (q - 1) * 16 / GK; i < q * 16 / GK; ++i) yp[i] = fmaf(s, acc[(t & 1) ^ 1][i], yp[i]);
                    }
                    request((grp * 2 * MB + t) * R + q, req, stage ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
    };

    int stage = 0;                                         // of the A operands of the next unit
    constexpr bool APART = qg_codes_slices_apart(GPS_, MB, TN, KW);
    auto slices_at = [&]() { return APART ? 2 * CHUNK * 1024 : (stage ^ 1) * CHUNK * 1024; };
    // End of a block's units in this workgroup: the whole sum to Y, a part of it to this part's place
    // among the partial results.
    auto finish = [&]() {
        if constexpr (SHORT) {
#pragma unroll
            for (int i = 0; i < 16; ++i) y[2 * MB - 1][i] = fmaf(sc[1][1], acc[1][i], y[2 * MB - 1][i]);
        } else {
#pragma unroll
            for (int k = 0; k < 2 * MB; ++k) fold(k);
        }
        // The sum over the k-slices of a tile, in slice order.  Four slices (blocks of 32 rows) share it: slice o takes OWN quads of the rows (a
        // quad: 8 rows x 32 outputs, four registers) and is handed the others' parts of those.  Of two slices slice 0 takes all, 32 rows at
        // a time.  (us, slice 0 | shares.  Four slices: 10135 x 640 3-bit g64 M = 11 6.9 | 6.4, 7146 x 2720 2-bit g32 M = 122 17.4 | 16.3, 13824 x
        // 5120 3-bit g64 M = 37 20.0 | 19.7, 149 products of 5 ... 128 rows 0.98 of the time.  Two: 24 products 1.006, and registers that the loop
        // wants: 21663 x 7680 4-bit g64 M = 59, 19 spilled, 40.0 | 43.0, 21060 x 3712 2-bit g64 M = 44 22.3 | 22.9.)
        constexpr bool SHARED = KW == 4;
        constexpr int OWN = 8 / KW;
        static_assert(KW == 2 || (SHARED && MB == 1), "slices of a workgroup");
        if constexpr (!APART) __syncthreads();               // every wavefront has read the unit's operands
        if constexpr (SHARED) {
            float *red = (float *)(smem + slices_at()) + tn * ((KW - 1) * 32 * 64) + lane;
#pragma unroll
            for (int o = 0; o < KW; ++o) {
                if (o == kw) continue;
                float *dst = red + (o * (KW - 1) + (kw < o ? kw : kw - 1)) * (OWN * 4 * 64);
#pragma unroll
                for (int i = 0; i < OWN * 4; ++i) dst[i * 64] = y[(o * OWN + i / 4) % 2][4 * ((o * OWN + i / 4) / 2) + i % 4];
            }
            __syncthreads();
#pragma unroll
            for (int o = 0; o < KW; ++o) {
                if (o != kw) continue;
                const float *src = red + o * (KW - 1) * (OWN * 4 * 64);
#pragma unroll
                for (int i = 0; i < OWN * 4; ++i) {
                    float &mine = y[(o * OWN + i / 4) % 2][4 * ((o * OWN + i / 4) / 2) + i % 4];
                    float sum = o == 0 ? mine : src[i * 64];
#pragma unroll
                    for (int j = 1; j < KW; ++j) sum += j == o ? mine : src[((j < o ? j : j - 1) * OWN * 4 + i) * 64];
                    mine = sum;
                }
            }
        } else {
            float *red = (float *)(smem + slices_at()) + lane;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                if (mb > 0) __syncthreads();
                if (kw > 0) {
                    float *dst = red + ((kw - 1) * TN + tn) * (32 * 64);
#pragma unroll
                    for (int i = 0; i < 32; ++i) dst[i * 64] = y[2 * mb + i / 16][i % 16];
                }
                __syncthreads();
                if (kw == 0) {
#pragma unroll
                    for (int j = 1; j < KW; ++j) {
                        const float *src = red + ((j - 1) * TN + tn) * (32 * 64);
#pragma unroll
                        for (int i = 0; i < 32; ++i) y[2 * mb + i / 16][i % 16] += src[i * 64];
                    }
                }
            }
        }
        // SHARED: body(qd) for every quad 2 band + pq of the tile that this slice has
        auto own_quads = [&](auto body) {
#pragma unroll
            for (int o = 0; o < KW; ++o) {
                if (o != kw) continue;
#pragma unroll
                for (int i = 0; i < OWN; ++i) body(o * OWN + i);
            }
        };
        const int tb = tiles_of(b), z = b - tb * A.zblocks, m0 = z * ROWS;
        const int tile = tb * TN + tn;
        int seg, nseg;
        if (A.ranges > 0) {
            seg = wg - b * A.ranges;
            nseg = A.ranges;
        } else {
            const int first = b * A.units / A.quota;
            seg = wg - first;
            nseg = ((b + 1) * A.units - 1) / A.quota - first + 1;
        }
        // Register i of an accumulator is row 8 (i / 4) + 4 half + i % 4 of its block: bands of eight rows,
        // a quad of registers each.  Stores quad (4 rows x 32 outputs, lane = row half and output) to Y.
        const int rows_left = A.M - m0;
        const int n0 = tile * QG_WAVE + row;
        const bool whole_tile = (tile + 1) * QG_WAVE <= A.N;
        auto store_y = [&](int r0, int pq, const float *v) {
            float *o = A.Y + (size_t)(m0 + r0 + 4 * half) * A.N + n0 + 32 * pq;
            if (whole_tile && r0 + 8 <= rows_left) {           // uniform: no test per lane
#pragma unroll
                for (int j = 0; j < 4; ++j) o[(size_t)j * A.N] = v[j];
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (r0 + 4 * half + j < rows_left && n0 + 32 * pq < A.N) o[(size_t)j * A.N] = v[j];
            }
        };
        constexpr int QUADS = 8 * MB;                          // quad 8 mb + 2 band + pq of a tile
        if (nseg == 1) {
            if constexpr (SHARED) {
                if (tile >= A.tiles) return;
                own_quads([&](int qd) {
                    const int r0 = 8 * (qd / 2);
                    if (r0 < rows_left) store_y(r0, qd % 2, &y[qd % 2][4 * (qd / 2)]);
                });
            } else {
                if (kw > 0 || tile >= A.tiles) return;
#pragma unroll
                for (int qd = 0; qd < QUADS; ++qd) {
                    const int r0 = 8 * (qd / 2), k = 2 * (qd / 8) + qd % 2;
                    if (r0 < rows_left) store_y(r0, qd % 2, &y[k][4 * ((qd / 2) % 4)]);
                }
            }
            return;
        }
        // A part of the sum, for add_parts or (fused) for the workgroup that comes last: every workgroup
        // writes its part and counts itself in; the one that finds the others there adds all parts in
        // the order of K (so the bits do not depend on who it is) and stores Y.  Those parts are written
        // and read past the caches of the chip's dies (sc1), and written before they are counted
        // (s_waitcnt); nobody waits for anybody.
        constexpr int SC1 = 16;
        const int bands = (A.M + 7) / 8;
        auto part_of = [&](int sg) {
            const int mine = (rows_left + 7) / 8;
            return buffer_of(A.partial + (((size_t)sg * A.tiles + tile) * bands + m0 / 8) * 2048, (mine < 4 * MB ? mine : 4 * MB) * 2048);
        };
        auto quad_of = [&](int qd) {
            const float *v = &y[2 * (qd / 8) + qd % 2][4 * ((qd / 2) % 4)];
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            return u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
        };
        if constexpr (!FUSED) {
            if ((!SHARED && kw > 0) || tile >= A.tiles) return;
            const rsrc_t part = part_of(seg);                  // (bands past M fall outside the buffer and are dropped)
            if constexpr (SHARED) {
                own_quads([&](int qd) { __builtin_amdgcn_raw_buffer_store_b128(quad_of(qd), part, lane16 + qd * 1024, 0, 0); });
            } else {
#pragma unroll
                for (int qd = 0; qd < QUADS; ++qd) __builtin_amdgcn_raw_buffer_store_b128(quad_of(qd), part, lane16 + qd * 1024, 0, 0);
            }
            return;
        } else {
        bool last = false;
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        if constexpr (SHARED) {
            if (tile < A.tiles) {
                const rsrc_t part = part_of(seg);
                own_quads([&](int qd) { __builtin_amdgcn_raw_buffer_store_b128(quad_of(qd), part, lane16 + qd * 1024, 0, SC1); });
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            __syncthreads();                                   // all slices' quads are written, and the sums have been read
        }
        if (kw == 0 && tile < A.tiles) {
            if constexpr (!SHARED) {
                const rsrc_t part = part_of(seg);
#pragma unroll
                for (int qd = 0; qd < QUADS; ++qd) __builtin_amdgcn_raw_buffer_store_b128(quad_of(qd), part, lane16 + qd * 1024, 0, SC1);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
            uint32_t before = 0;
            if (lane == 0)
                before = __hip_atomic_fetch_add(A.arrived + (size_t)tile * A.zblocks + z, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = (int)__builtin_amdgcn_readfirstlane(before) + 1 == nseg;
        }
        {
            // slice 0 tells the others, in a word that is read no more (SHARED: by nobody, else by slice 0 of its own tile alone)
            uint32_t *flag = (uint32_t *)(smem + slices_at()) + (SHARED ? tn : tn * (32 * 64));
            if (kw == 0 && lane == 0) *flag = last;
            __syncthreads();
            last = __builtin_amdgcn_readfirstlane(*flag) != 0;
        }
        if (!last || tile >= A.tiles) return;
        constexpr int SHARE = QUADS / KW, AT_ONCE = SHARE < 2 ? SHARE : 2;
        static_assert(QUADS % KW == 0 && SHARE % AT_ONCE == 0, "quads per wavefront");
        for (int q0 = kw * SHARE; q0 < (kw + 1) * SHARE; q0 += AT_ONCE) {
            u32x4 v[AT_ONCE][QG_FUSED_SEGMENTS];
#pragma unroll
            for (int sg = 0; sg < QG_FUSED_SEGMENTS; ++sg)
                if (sg < nseg) {
                    const rsrc_t part = part_of(sg);
#pragma unroll
                    for (int i = 0; i < AT_ONCE; ++i) v[i][sg] = __builtin_amdgcn_raw_buffer_load_b128(part, lane16 + (q0 + i) * 1024, 0, SC1);
                }
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) {
                float t[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] = __uint_as_float(v[i][0][j]);
#pragma unroll
                for (int sg = 1; sg < QG_FUSED_SEGMENTS; ++sg)
                    if (sg < nseg) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) t[j] += __uint_as_float(v[i][sg][j]);
                    }
                const int r0 = 8 * ((q0 + i) / 2);
                if (r0 < rows_left) store_y(r0, (q0 + i) % 2, t);
            }
        }
        }
    };

    // Unit u is computed from registers and LDS filled while unit u - 1 was; two register sets and two
    // LDS stages take turns.  Everything requested during a unit has arrived at the barrier that ends
    // it.  The last unit requests itself again (no branches in the loop body, nothing used).
    StepRegs ra, rb;
    auto arrive = [&](StepRegs &r) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < L; ++i) asm volatile("" : "+v"(r.v[i].x), "+v"(r.v[i].y), "+v"(r.v[i].z), "+v"(r.v[i].w));
#pragma unroll
        for (int g = 0; g < GPS; ++g) asm volatile("" : "+v"(r.s[g]));
        asm volatile("" : "+v"(r.zw));
        __syncthreads();
    };
    auto unit = [&](StepRegs &use, StepRegs &req) {
        if constexpr (SELF) store_x(stage);
        arrive(use);
        const uint32_t step = it * KW + kw;
        const bool last = u + 1 >= u1, ends = it + 1 >= A.units;
        const int nit = last ? it : ends ? 0 : it + 1;
        if (ends && !last) aim_block(b + 1);
        aim(nit);
        if constexpr (SELF) {
            if (!last) load_x();
        }
        if constexpr (SHORT) compute_short(use, step, stage, req);
        else compute(use, step, stage, req);
        stage ^= 1;
        if (ends || last) {
            finish();
            if (!last) {
                reset();
                ++b;
            }
        }
        it = nit;
        ++u;
    };
    reset();
    aim_block(b);
    aim(it);
#pragma unroll
    for (int t = 0; t < NLOAD + NDMA; ++t) request(t, ra, 0);
    if constexpr (SELF) load_x();
    while (u < u1) {
        unit(ra, rb);
        if (u >= u1) break;
        unit(rb, ra);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no copy into LDS outlives the workgroup
}

template <int BITS, int GPS, int MB, int TN, int KW, int HOW>
int codes_launch(const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query)
{
    static_assert(qg_codes_lds(GPS, MB, TN, KW) <= QG_LDS_BYTES, "LDS of a workgroup");
    static_assert(qg_codes_slices_apart(GPS, MB, TN, KW) || (KW - 1) * TN * 32 * 256 <= qg_codes_stages(GPS, MB, KW) / 2, "slices in a stage");
    constexpr size_t lds = qg_codes_lds(GPS, MB, TN, KW);
    const void *f = (const void *)gemm_codes<BITS, GPS, MB, TN, KW, HOW>;
    if (query) {
        *query = {f, TN * KW * 64, lds};
        return QG_OK;
    }
    // dynamic LDS above 64 KB has to be asked for, once per device (devices past the table: every time;
    // two threads at once ask twice)
    static std::atomic<bool> prepared[64];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
    if (dev < 0 || !prepared[dev].load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
            (void)hipGetLastError();
            return QG_ERR_DEVICE;
        }
        if (dev >= 0) prepared[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((gemm_codes<BITS, GPS, MB, TN, KW, HOW>), dim3((unsigned)workgroups), dim3(TN * KW * 64), lds, st, A);
    return QG_OK;
}

template <int BITS, int GPS, int MB, int KW>
int codes_launch_how(const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query)
{
    if (A.self) {
        if constexpr (MB == 1 && GPS <= 4) return codes_launch<BITS, GPS, MB, 8 / KW, KW, QG_CODES_SELF>(A, workgroups, st, query);
        return QG_ERR_UNSUPPORTED;
    }
    return A.fused ? codes_launch<BITS, GPS, MB, 8 / KW, KW, QG_CODES_FUSED>(A, workgroups, st, query)
                   : codes_launch<BITS, GPS, MB, 8 / KW, KW, QG_CODES_PREPARED>(A, workgroups, st, query);
}

template <int BITS, int GPS>
int codes_launch_shape(int mb, const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query)
{
    constexpr int FEW = qg_codes_kw(GPS, 1, false), MANY = qg_codes_kw(GPS, 1, true);
    if (mb == 2) return codes_launch_how<BITS, GPS, 2, qg_codes_kw(GPS, 2, true)>(A, workgroups, st, query);
    return A.kw == FEW ? codes_launch_how<BITS, GPS, 1, FEW>(A, workgroups, st, query)
                       : codes_launch_how<BITS, GPS, 1, MANY>(A, workgroups, st, query);
}

template <int BITS>
int codes_launch_any(int gps, int mb, const QgCodesArgs &A, int workgroups, hipStream_t st, QgKernelInfo *query)
{
    switch (gps) {
    case 0: return codes_launch_shape<BITS, 0>(mb, A, workgroups, st, query);
    case 1: return codes_launch_shape<BITS, 1>(mb, A, workgroups, st, query);
    case 2: return codes_launch_shape<BITS, 2>(mb, A, workgroups, st, query);
    case 4:
        if constexpr (BITS != 3) return codes_launch_shape<BITS, 4>(mb, A, workgroups, st, query);
        return QG_ERR_UNSUPPORTED;
    case 8:
        if constexpr (BITS == 4) return codes_launch_shape<BITS, 8>(mb, A, workgroups, st, query);
        return QG_ERR_UNSUPPORTED;
    default: return QG_ERR_UNSUPPORTED;
    }
}

template <int BITS>
void codes_prepare(const QgPrepArgs &P, int rows_padded, hipStream_t st)
{
    hipLaunchKernelGGL(prepare_x<BITS>, dim3((unsigned)P.steps_padded, (unsigned)rows_padded / 32), dim3(32 * 128 / (BITS == 2 ? 16 : 8)), 0, st, P);
}

}  // namespace
#endif
