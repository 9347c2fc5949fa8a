// The small-M product of 3-bit groups of 32 weights, in the arithmetic of the GEMV: X as 32-bit fixed point, sums of
// codes times digits exact in int32, scales in fp32.  (The bf16 kernels of qg_gemm_small do not take these groups.)
//
// X is converted once per call (prepare_rows_i8): per row and unit of 128 k one power of two brings the largest |x|
// below 2^30, the rounded integers are cut into four signed base-256 digits, and the digits of eight rows are the 32 rows
// of an A operand of v_mfma_i32_32x32x32_i8, whose 32 k are one group.  The B operand is q - z as bytes, 32 outputs: an
// accumulator then holds, for an output and four of the eight rows, the four digit sums of a group in neighbouring
// registers, which make one fp32 number that enters y with the group's scale.  No zero-point is left to subtract.
//
// A wavefront owns a tile of 64 outputs (device layout, lane = output; one v_permlane32_swap per pair of words turns that
// into the operand layout) and NB blocks of eight rows, and goes through a range of K; the wavefronts of a workgroup are
// k-slices of one tile and meet in LDS.  A operands come straight from L2: 1 KB per group and block of rows, against 1 KB
// of codes and scales.
//
// What bounds it: instruction issue, 35 vector instructions per group and tile for the codes and 48 per block of eight
// rows for the digit sums (beside 2 matrix instructions), and the operands' way from L2 under them.
// Measured (us per call; before: a matrix-vector product per row, 16 rows to a launch): 10486 x 16608 M = 15 443 -> 46,
// 4096 x 4096 M = 16 16.2 -> 11.7, M = 128 120 -> 29.5, 13824 x 5120 M = 37 145 -> 53; error against 64 bits (2-norm) 1.7e-7
// to 3.3e-7 -> 0.7e-7 to 1e-7.
#include "qg_common.h"
#include "qg_mma.h"

struct QgRowsI8Args {
    const uint4 *codes;        // [tile][unit][plane][lane]
    const float *scales;       // [tile][group][lane]
    const uint32_t *zeros;     // [tile][zero word][lane]
    const int4 *Aop;           // [block of 8 rows][group][lane] (prepare_rows_i8)
    const float *inverse;      // [block of 8 rows][unit][row parity][4]: what the integers of a row are multiplied by
    float *out;                // [range][M][N]
    int M, N, tiles, ngroups, zwords, units, units_padded;     // units of 128 k in K, and as stored
    int per_wave;              // units per wavefront
};

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
constexpr int UNIT_K = 128, SLICES = 4;

// A wavefront converts eight rows x one unit: lane 8 r + i holds k 16 i ... 16 i + 15 of row r.
__global__ __launch_bounds__(64) void prepare_rows_i8(const float *__restrict__ X, int M, int K, int units, int4 *__restrict__ Aop,
                                                      float *__restrict__ inverse)
{
    const int u = blockIdx.x, rb = blockIdx.y, row = threadIdx.x >> 3, i = threadIdx.x & 7;
    const int m = rb * 8 + row, k = u * UNIT_K + 16 * i;
    float x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = 0.0f;
    if (m < M && k < K) {                                  // (K is a whole number of 32)
        const float4 *src = (const float4 *)(X + (size_t)m * K + k);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 v = src[j];
            x[4 * j] = v.x; x[4 * j + 1] = v.y; x[4 * j + 2] = v.z; x[4 * j + 3] = v.w;
        }
    }
    uint32_t most = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint32_t bits = __float_as_uint(x[j]) & 0x7fffffffu;
        most = bits > most ? bits : most;
    }
#pragma unroll
    for (int off = 1; off < 8; off *= 2) {
        const uint32_t other = (uint32_t)__shfl_xor((int)most, off, 64);
        most = other > most ? other : most;
    }
    // |x| < 2^(e - 126): times 2^(156 - e) below 2^30; below 2^-96 less precise rather than out of range
    const int e = (int)(most >> 23);
    const int up = 283 - e < 253 ? 283 - e : 253;         // biased exponent of the factor
    const float factor = __uint_as_float((uint32_t)up << 23);
    uint32_t d[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) d[j] = ((uint32_t)__float2int_rn(x[j] * factor) + 0x00808080u) ^ 0x00808080u;
    uint32_t digit[4][4];                                  // [digit][dword]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t lo01 = __builtin_amdgcn_perm(d[4 * q + 1], d[4 * q], 0x05010400u), hi01 = __builtin_amdgcn_perm(d[4 * q + 1], d[4 * q], 0x07030602u);
        const uint32_t lo23 = __builtin_amdgcn_perm(d[4 * q + 3], d[4 * q + 2], 0x05010400u), hi23 = __builtin_amdgcn_perm(d[4 * q + 3], d[4 * q + 2], 0x07030602u);
        digit[0][q] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        digit[1][q] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        digit[2][q] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        digit[3][q] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
    }
    int4 *to = Aop + ((size_t)(rb * units + u) * 4 + i / 2) * 64 + (i & 1) * 32 + row * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) to[q] = make_int4((int)digit[q][0], (int)digit[q][1], (int)digit[q][2], (int)digit[q][3]);
    // NaN or infinity among a row's values makes the row of Y NaN
    if (i == 0)
        inverse[((size_t)rb * units + u) * 8 + (row & 1) * 4 + row / 2] = most >= 0x7f800000u ? __uint_as_float(0x7fc00000u) : __uint_as_float((uint32_t)(254 - up) << 23);
}

template <int NB>
__global__ __launch_bounds__(SLICES * 64, NB == 1 ? 3 : 2) void gemm_rows_i8(const QgRowsI8Args A)
{
    __shared__ float red[SLICES - 1][8 * NB][64];
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x, rb0 = blockIdx.z * NB;
    const int u0 = (blockIdx.y * SLICES + wave) * A.per_wave;
    const int u1 = u0 + A.per_wave < A.units ? u0 + A.per_wave : A.units;
    const int blocks = (A.M + 7) / 8;

    struct Unit {
        uint4 v[3];
        float sP[4], sQ[4];            // scales of outputs col, 32 + col
        uint32_t zP, zQ;
    };
    // (the A operands of a group are asked for as soon as the unit before has used its own: three groups ahead)
    i32x4 a[4][NB];
    float4 inv[NB];
    const char *a_from[NB];
    const float *inv_from[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int rb = rb0 + nb < blocks ? rb0 + nb : blocks - 1;          // (the last block again: not stored)
        a_from[nb] = (const char *)(A.Aop + (size_t)rb * A.units * 4 * 64);
        inv_from[nb] = A.inverse + (size_t)rb * A.units * 8;
    }
    auto load_a = [&](int u, int j) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) a[j][nb] = *(const i32x4 *)(a_from[nb] + ((size_t)u * 4 + j) * 1024 + lane * 16);
    };
    auto load_inv = [&](int u) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) inv[nb] = *(const float4 *)(inv_from[nb] + (size_t)u * 8 + half * 4);
    };
    auto load = [&](int u, Unit &r) {
#pragma unroll
        for (int p = 0; p < 3; ++p) r.v[p] = A.codes[((size_t)tile * A.units_padded + u) * 3 * 64 + p * 64 + lane];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // (groups past K meet zeros)
            const int g = 4 * u + j < A.ngroups ? 4 * u + j : A.ngroups - 1;
            const float *s = A.scales + ((size_t)tile * A.ngroups + g) * 64 + col;
            r.sP[j] = s[0];
            r.sQ[j] = s[32];
        }
        const uint32_t *z = A.zeros + ((size_t)tile * A.zwords + u / 2) * 64 + col;
        r.zP = z[0] >> (16 * (u & 1));
        r.zQ = z[32] >> (16 * (u & 1));
    };
    float y[NB][2][4];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int pq = 0; pq < 2; ++pq)
#pragma unroll
            for (int i = 0; i < 4; ++i) y[nb][pq][i] = 0.0f;
    const i32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    auto compute = [&](const Unit &r, int next) {
        float part[NB][2][4];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int pq = 0; pq < 2; ++pq)
#pragma unroll
                for (int i = 0; i < 4; ++i) part[nb][pq][i] = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // a cell: words 0 and 1 hold codes 0-15, word 2 and the spare bits of all three codes 16-31
            const uint32_t w0 = word_of(r.v[0], j), w1 = word_of(r.v[1], j), w2 = word_of(r.v[2], j);
            const uint32_t w3 = ((w0 >> 6) & 0x03030303u) | ((w1 >> 4) & 0x0c0c0c0cu) | ((w2 >> 2) & 0x30303030u);
            const auto s0 = __builtin_amdgcn_permlane32_swap(w0, w2, false, false), s1 = __builtin_amdgcn_permlane32_swap(w1, w3, false, false);
#pragma unroll
            for (int pq = 0; pq < 2; ++pq) {
                const uint32_t z = ((pq ? r.zQ : r.zP) >> (4 * j)) & 15u, zb = __builtin_amdgcn_perm(z, z, 0u);
                // bytes q - z: the borrow of a byte stops at its bit 7
                auto minus_z = [&](uint32_t w) { return (int)((((w & 0x07070707u) | 0x80808080u) - zb) ^ 0x80808080u); };
                const i32x4 b = {minus_z(s0[pq]), minus_z(s0[pq] >> 3), minus_z(s1[pq]), minus_z(s1[pq] >> 3)};
                float s = pq ? r.sQ[j] : r.sP[j];
                asm volatile("" : "+v"(s));
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const i32x16 t = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[j][nb], b, zero16, 0, 0, 0);
                    // digits of row 2 i + half: the lower three together stay below 32 * 7 * 2^7 * (2^16 + 2^8 + 1) < 2^31
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int low = t[4 * i] + (t[4 * i + 1] << 8) + (t[4 * i + 2] << 16);
                        const float sum = fmaf((float)t[4 * i + 3], 16777216.0f, (float)low);
                        part[nb][pq][i] = fmaf(s, sum, part[nb][pq][i]);
                        // (one accumulator after the other: the compiler otherwise holds those of several groups and spills)
                        asm volatile("" : "+v"(part[nb][pq][i]));
                    }
                    asm volatile("" ::: "memory");
                }
            }
            load_a(next, j);
            asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const float f[4] = {inv[nb].x, inv[nb].y, inv[nb].z, inv[nb].w};
#pragma unroll
            for (int pq = 0; pq < 2; ++pq)
#pragma unroll
                for (int i = 0; i < 4; ++i) y[nb][pq][i] = fmaf(f[i], part[nb][pq][i], y[nb][pq][i]);
        }
        load_inv(next);
    };
    if (u0 < u1) {
        Unit ra, rb;
        load(u0, ra);
#pragma unroll
        for (int j = 0; j < 4; ++j) load_a(u0, j);
        load_inv(u0);
        for (int u = u0; u < u1; u += 2) {
            const int n1 = u + 1 < u1 ? u + 1 : u, n2 = u + 2 < u1 ? u + 2 : u;
            load(n1, rb);
            compute(ra, n1);
            if (u + 1 >= u1) break;
            load(n2, ra);
            compute(rb, n2);
        }
    }
    // k-slices, in the order of K
    if (wave > 0) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int pq = 0; pq < 2; ++pq)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[wave - 1][(nb * 2 + pq) * 4 + i][lane] = y[nb][pq][i];
    }
    __syncthreads();
    if (wave > 0) return;
    float *out = A.out + (size_t)blockIdx.y * A.M * A.N;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int pq = 0; pq < 2; ++pq)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float t = y[nb][pq][i];
#pragma unroll
                for (int s = 0; s < SLICES - 1; ++s) t += red[s][(nb * 2 + pq) * 4 + i][lane];
                const int m = (rb0 + nb) * 8 + 2 * i + half, n = tile * 64 + 32 * pq + col;
                if (m < A.M && n < A.N) out[(size_t)m * A.N + n] = t;
            }
}

struct RowsI8Plan {
    int blocks, nb, zblocks, units, splits, per_wave;
    size_t inverse_off, partial_off, total;
};
RowsI8Plan rows_i8_plan(const QgLayout &L, int M)
{
    RowsI8Plan P;
    P.blocks = (M + 7) / 8;
    P.nb = P.blocks <= 1 ? 1 : P.blocks <= 2 ? 2 : 4;
    P.zblocks = (P.blocks + P.nb - 1) / P.nb;
    P.units = (int)((L.K + UNIT_K - 1) / UNIT_K);
    // two wavefronts per SIMD, each with two units of K at least
    const int64_t waves = L.tiles * P.zblocks * SLICES, want = (int64_t)qg_compute_units() * 8;
    int most = P.units / (2 * SLICES) < 8 ? P.units / (2 * SLICES) : 8;
    if (most < 1) most = 1;
    int splits = (int)((want + waves - 1) / waves);
    if (splits > most) splits = most;
    P.per_wave = (P.units + splits * SLICES - 1) / (splits * SLICES);
    P.splits = (P.units + P.per_wave * SLICES - 1) / (P.per_wave * SLICES);
    P.inverse_off = (size_t)P.blocks * P.units * 4 * 1024;
    P.partial_off = qg_round_up(P.inverse_off + (size_t)P.blocks * P.units * 8 * sizeof(float), QG_SECTION_ALIGN);
    // (as many parts as any device's plan may take; a K of up to 1920 is in one)
    P.total = qg_round_up(P.partial_off + (most > 1 ? (size_t)most * M * L.N * sizeof(float) : 0), QG_SECTION_ALIGN);
    return P;
}

}  // namespace

// Whether the kernel takes a layout: 3-bit groups of one cell.
bool qg_rows_i8_takes(const QgLayout &L) { return L.bits == 3 && L.group == 32 && L.K <= (1 << 20) && L.N <= (1 << 22); }
size_t qg_rows_i8_bytes(const QgLayout &L, int M) { return rows_i8_plan(L, M).total; }
int qg_rows_i8_splits(const QgLayout &L, int M) { return rows_i8_plan(L, M).splits; }

// Kernels' time of a call, adding the parts included: a unit's instructions at 1.78 times the time they issue in, as
// measured from 4096 x 4096 to 10486 x 16608 (29.5, 53.4, 46.0 us for 29.6, 53.1, 46.0), and on a chip that is not full the
// chain of its blocks of rows, one after the other: 1.6, 2.0 and 3.4 us (100 products of less than a wavefront per
// SIMD, 64 to 22000 outputs and inputs: 6 % off; as for one block, 1.6, 75 x 1536 M = 18 was priced at 9.4 us for 14.3).
double qg_rows_i8_us(const QgLayout &L, int M)
{
    const RowsI8Plan P = rows_i8_plan(L, M);
    const double unit = P.nb == 1 ? 0.55 : P.nb == 2 ? 0.87 : 1.5, least = P.nb == 1 ? 0.9 : P.nb == 2 ? 1.1 : 1.9;
    const double waves = (double)L.tiles * P.zblocks * P.splits * SLICES / (4.0 * qg_compute_units());
    const double busy = unit * waves > least ? unit * waves : least;
    return 4.6 + 1.78 * P.per_wave * busy + (P.splits > 1 ? 2.0 + 1.5e-6 * P.splits * M * L.N : 0.0);
}

// Enqueues the conversion and the product; *partial: where the parts of the sum are if there are several.
int qg_rows_i8(const void *packed, const QgLayout &L, const float *X, int M, float *Y, void *workspace, hipStream_t st, float **partial)
{
    const RowsI8Plan P = rows_i8_plan(L, M);
    char *ws = (char *)workspace;
    const char *base = (const char *)packed;
    *partial = (float *)(ws + P.partial_off);
    QgRowsI8Args A;
    A.codes = (const uint4 *)(base + L.codes_off);
    A.scales = (const float *)(base + L.scales_off);
    A.zeros = (const uint32_t *)(base + L.zeros_off);
    A.Aop = (const int4 *)ws;
    A.inverse = (const float *)(ws + P.inverse_off);
    A.out = P.splits > 1 ? *partial : Y;
    A.M = M;
    A.N = (int)L.N;
    A.tiles = (int)L.tiles;
    A.ngroups = (int)L.ngroups;
    A.zwords = (int)L.zwords;
    A.units = P.units;
    A.units_padded = (int)L.units;
    A.per_wave = P.per_wave;
    hipLaunchKernelGGL(prepare_rows_i8, dim3((unsigned)P.units, (unsigned)P.blocks), dim3(64), 0, st, X, M, (int)L.K, P.units, (int4 *)ws, (float *)(ws + P.inverse_off));
    if (qg_launch_status() != QG_OK) return QG_ERR_DEVICE;
    const dim3 grid((unsigned)L.tiles, (unsigned)P.splits, (unsigned)P.zblocks);
    if (P.nb == 1) hipLaunchKernelGGL(gemm_rows_i8<1>, grid, dim3(SLICES * 64), 0, st, A);
    else if (P.nb == 2) hipLaunchKernelGGL(gemm_rows_i8<2>, grid, dim3(SLICES * 64), 0, st, A);
    else hipLaunchKernelGGL(gemm_rows_i8<4>, grid, dim3(SLICES * 64), 0, st, A);
    return qg_launch_status();
}
