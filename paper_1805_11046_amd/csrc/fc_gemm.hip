// Fully connected products (Section 4: Y = X W, g_{l-1} = g_l W^T; Sections 1, 7: g_W = X^T g_l with the 16-bit copy
// of g_l) on the int8 MFMAs, operands read where they lie: nothing is transposed or padded in memory first.
//
// Every product is rows x cols over a reduction:
//   forward   rows m, cols n, reduction k:  A = X  [m][k], B = W   [k][n]
//   dgrad     rows m, cols k, reduction n:  A = dY [m][n], B = W   [k][n]
//   wgrad     rows k, cols n, reduction m:  A = X  [m][k], B = dY16[m][n] (two byte planes, s = 256*hi + lo + 128)
// An operand whose reduction index is the fast one ("RF") gives a lane its 16 MFMA bytes with one 16-byte load.  An
// operand whose reduction index is the slow one ("RS") is read as dwords, four neighbouring columns of one reduction
// index each; 4x4 byte transposes (v_perm) turn 16 of them into the 16-byte pieces of four columns.  The columns
// 4c .. 4c+3 of a lane group therefore go to four different MFMA tiles, and a lane ends up with four neighbouring
// results of a row, which leave as one 16-byte store.
//
// Ragged sizes cost no padding and no access outside a tensor: a group of columns (rows) that would hang over the
// edge starts at the last full group instead (its results are computed twice, with the same value), and a piece of
// the reduction that would hang over the end starts earlier with the entries already counted masked to zero in
// both operands.  With masked entries zero, sum (a-za)(b-zb) = sum ab - zb sum a - za sum b + red za zb holds
// for the real reduction length.
//
// Three kernels (times: back to back on one MI355X, M x N x K, against the general kernel that served every FC call before):
//   fc_direct  operands go from memory to registers, no LDS in the main loop; the wavefronts of a workgroup share a
//              tile of 32x64 (wgrad 64x64) results and split its reduction, or own a tile each.  Bound by latency
//              (launch, one or two dependent loads, the fold through LDS): 64x128x256 takes 3.9 / 3.9 / 6.0 us for
//              forward / dgrad / wgrad (18.7 / 12.2 / 8.0 before), 256x1000x512 4.7 / 5.2 / 6.8 (23.9 / 15.8 / 19.7), the
//              forward and dgrad of 512x2048x2048 10.7 and 15.0.  Few results and a long reduction: slices of it in
//              workgroups of their own and fc_fold behind them.
//   fc_dma     matrices of aligned rows, many tiles: operands go to LDS without registers (see there).
//   fc_tile    the same sizes at any address and pitch: 128x128 tiles, K-steps of 64 through double-buffered LDS with two
//              register sets of prefetch.  65 / 59 / 112 us at 2048x4096x4096 (1002 / 1777 / 473 before), 1.0 - 1.2 POP/s.
// Measured and dropped: prefetching the next K-step in fc_direct (more registers, fewer wavefronts: 7.5 -> 8.4 us at
// 1024^3), K-steps of 128 in fc_tile with one or two register sets (whole 128-byte lines per row: 68 / 61 and
// 68 / 65 us against 70 / 64 on the same box, 3000x333x2777 30 -> 38).
#include "q8t_common.h"
#include "q8t_internal.h"
#include "gemm_core.h"

namespace {

using q8t_gemm::swz;
using q8t_gemm::v4i;

enum { FWD = 0, DGRAD = 1, WGRAD = 2 };

struct FcArgs {
    const int8_t *a;
    const void *b;
    const q8t_qparams *qa, *qb;
    int rows, cols, red;
    int lda, ldb;        // elements between neighbours along the slow index
    float *out;          // nullable
    void *acc;           // nullable: int32 (forward, dgrad) or int64 (wgrad)
    int64_t *partial;    // not NULL: a slice of the reduction leaves its share of the results here, [slice][rows][cols]
    int slice;           // K-steps per slice
    int vec;             // float results leave in 16-byte stores
    int tn, tiles;       // column tiles, all tiles
};

__device__ __forceinline__ uint4 ld16(const void *p)
{
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}
__device__ __forceinline__ uint2 ld8(const void *p)
{
    uint2 v;
    __builtin_memcpy(&v, p, 8);
    return v;
}
__device__ __forceinline__ uint32_t ld4(const void *p)
{
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}
__device__ __forceinline__ int dot4_ones(uint32_t v, int acc) { return __builtin_amdgcn_sdot4((int)v, 0x01010101, acc, false); }

// in[i] = columns 0..3 of reduction index i; out[j] = reduction indices 0..3 of column j
__device__ __forceinline__ void transpose4x4(uint32_t i0, uint32_t i1, uint32_t i2, uint32_t i3, uint32_t (&out)[4])
{
    const uint32_t t0 = __builtin_amdgcn_perm(i1, i0, 0x05010400);
    const uint32_t t1 = __builtin_amdgcn_perm(i1, i0, 0x07030602);
    const uint32_t t2 = __builtin_amdgcn_perm(i3, i2, 0x05010400);
    const uint32_t t3 = __builtin_amdgcn_perm(i3, i2, 0x07030602);
    out[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100);
    out[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302);
    out[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100);
    out[3] = __builtin_amdgcn_perm(t3, t1, 0x07060302);
}
// high / (re-centred) low bytes of four 16-bit codes
__device__ __forceinline__ uint32_t hi_bytes(const uint2 &v) { return __builtin_amdgcn_perm(v.y, v.x, 0x07050301); }
__device__ __forceinline__ uint32_t lo_bytes(const uint2 &v) { return __builtin_amdgcn_perm(v.y, v.x, 0x06040200) ^ 0x80808080u; }

// bytes first .. first+3 of a piece whose first `skip` bytes are masked out
__device__ __forceinline__ uint32_t keep_mask(int first, int skip)
{
    const int n = min(max(skip - first, 0), 4);
    return n == 4 ? 0u : 0xFFFFFFFFu << (8 * n);
}

struct Zero {
    int za, zb;
    float sc;
};
__device__ __forceinline__ Zero zero_points(const FcArgs &p)
{
    Zero z;
    z.za = p.qa->zero_point - (1 << (p.qa->bits - 1));
    z.zb = p.qb->zero_point - (1 << (p.qb->bits - 1));
    z.sc = p.qa->scale * p.qb->scale;
    return z;
}

// four neighbouring results of one row; v[j] the accumulators, rs / cs the byte sums of the row and the columns
// (wgrad: cs = 256 * sum hi + sum lo), red the entries of the reduction in them
template <int WHICH>
__device__ __forceinline__ void finish4(const FcArgs &p, const Zero &z, int red, int row, int col, const int (&hi)[4],
                                        const int (&lo)[4], int rs, const int (&cs)[4], const int (&cs1)[4])
{
    const int64_t o = (int64_t)row * p.cols + col;
    float f[4];
    if (WHICH != WGRAD) {
        const uint32_t kzz = (uint32_t)red * (uint32_t)z.za * (uint32_t)z.zb - (uint32_t)z.zb * (uint32_t)rs;
        int c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = (int)((uint32_t)hi[j] + kzz - (uint32_t)z.za * (uint32_t)cs[j]);   // fits 32 bits by contract
            f[j] = z.sc * (float)c[j];
        }
        if (p.partial) {
            int64_t *d = p.partial + (int64_t)blockIdx.y * p.rows * p.cols + o;
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = c[j];
            return;
        }
        if (p.acc) {
            int32_t *d = (int32_t *)p.acc + o;
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = c[j];
        }
    } else {
        const int64_t t = (int64_t)(128 - z.zb) * rs + (int64_t)red * z.za * (z.zb - 128);
        int64_t c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] = 256 * (int64_t)hi[j] + lo[j] + t - (int64_t)z.za * (256 * (int64_t)cs[j] + cs1[j]);
            f[j] = (float)((double)c[j] * (double)z.sc);
        }
        if (p.partial) {
            int64_t *d = p.partial + (int64_t)blockIdx.y * p.rows * p.cols + o;
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = c[j];
            return;
        }
        if (p.acc) {
            int64_t *d = (int64_t *)p.acc + o;
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = c[j];
        }
    }
    if (p.out) {
        float *d = p.out + o;
        if (p.vec) {
            *reinterpret_cast<float4 *>(d) = make_float4(f[0], f[1], f[2], f[3]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = f[j];
        }
    }
}

// ---- small products: no LDS in the main loop ---------------------------------------------------------------------
// KS wavefronts share a tile's reduction (K-steps of 64, dealt out round-robin); WAVES / KS tiles per workgroup.  Where the
// tiles are few and the reduction is long, blockIdx.y takes slices of it, and fc_fold adds them up.
template <int WHICH, int WAVES, int KS>
__global__ __launch_bounds__(WAVES * 64) void fc_direct(const FcArgs p)
{
    constexpr bool RSA = WHICH == WGRAD, RSB = WHICH != DGRAD;
    constexpr int PL = WHICH == WGRAD ? 2 : 1;
    constexpr int MT = RSA ? 4 : 2, TR = MT * 16;     // rows of a tile
    constexpr int UNITS = MT * 4;                     // (mt, j): a lane's groups of four results
    constexpr int TPB = WAVES / KS;
    __shared__ int s_rs[TPB][TR], s_cs[TPB][PL][64];
    __shared__ __attribute__((aligned(16))) int s_acc[KS > 1 ? WAVES * UNITS * 256 : 4];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kb = lane >> 4;
    const int sub = wave / KS, ks = wave % KS;
    for (int i = tid; i < TPB * TR; i += WAVES * 64) (&s_rs[0][0])[i] = 0;
    for (int i = tid; i < TPB * PL * 64; i += WAVES * 64) (&s_cs[0][0][0])[i] = 0;
    __syncthreads();
    const int tile = min((int)blockIdx.x * TPB + sub, p.tiles - 1);   // a surplus wavefront repeats the last tile
    const int m0 = (tile / p.tn) * TR, n0 = (tile % p.tn) * 64;

    // rows / columns of the lane's pieces
    const int8_t *pa[MT];
    if (RSA) {
        pa[0] = p.a + min(m0 + 4 * l16, p.rows - 4);
    } else {
#pragma unroll
        for (int i = 0; i < MT; ++i) pa[i] = p.a + (int64_t)min(m0 + i * 16 + l16, p.rows - 1) * p.lda;
    }
    const int col0 = min(n0 + 4 * l16, p.cols - 4);   // the lane's four columns, RF and RS alike
    const int8_t *pb8 = (const int8_t *)p.b;
    const int16_t *pb16 = (const int16_t *)p.b;

    v4i acc[PL][MT][4];
    int sa[MT], sb[PL][4];
#pragma unroll
    for (int h = 0; h < PL; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sb[h][j] = 0;
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[h][i][j] = (v4i){0, 0, 0, 0};
        }
#pragma unroll
    for (int i = 0; i < MT; ++i) sa[i] = 0;

    const int steps = (p.red + 63) >> 6;
    const int s0 = blockIdx.y * p.slice, s1 = min(steps, s0 + p.slice), red = min(s1 * 64, p.red) - s0 * 64;
    for (int s = s0 + ks; s < s1; s += KS) {
        const int kk = s * 64 + kb * 16, k1 = min(kk, p.red - 16), skip = kk - k1;
        uint4 af[MT], bf[PL][4];
        uint32_t ra[RSA ? 16 : 1], rb[RSB && PL == 1 ? 16 : 1];
        uint2 rb16[PL == 2 ? 16 : 1];
        // all loads of the step first
        if (RSA) {
#pragma unroll
            for (int i = 0; i < 16; ++i) ra[i] = ld4(pa[0] + (int64_t)(k1 + i) * p.lda);
        } else {
#pragma unroll
            for (int i = 0; i < MT; ++i) af[i] = ld16(pa[i] + k1);
        }
        if (PL == 2) {
#pragma unroll
            for (int i = 0; i < 16; ++i) rb16[i] = ld8(pb16 + (int64_t)(k1 + i) * p.ldb + col0);
        } else if (RSB) {
#pragma unroll
            for (int i = 0; i < 16; ++i) rb[i] = ld4(pb8 + (int64_t)(k1 + i) * p.ldb + col0);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) bf[0][j] = ld16(pb8 + (int64_t)(col0 + j) * p.ldb + k1);
        }
        if (RSA) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t o[4];
                transpose4x4(ra[4 * d], ra[4 * d + 1], ra[4 * d + 2], ra[4 * d + 3], o);
#pragma unroll
                for (int i = 0; i < MT; ++i) (&af[i].x)[d] = o[i];
            }
        }
        if (PL == 2) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t o[4];
                transpose4x4(hi_bytes(rb16[4 * d]), hi_bytes(rb16[4 * d + 1]), hi_bytes(rb16[4 * d + 2]), hi_bytes(rb16[4 * d + 3]), o);
#pragma unroll
                for (int j = 0; j < 4; ++j) (&bf[0][j].x)[d] = o[j];
                transpose4x4(lo_bytes(rb16[4 * d]), lo_bytes(rb16[4 * d + 1]), lo_bytes(rb16[4 * d + 2]), lo_bytes(rb16[4 * d + 3]), o);
#pragma unroll
                for (int j = 0; j < 4; ++j) (&bf[PL - 1][j].x)[d] = o[j];
            }
        } else if (RSB) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t o[4];
                transpose4x4(rb[4 * d], rb[4 * d + 1], rb[4 * d + 2], rb[4 * d + 3], o);
#pragma unroll
                for (int j = 0; j < 4; ++j) (&bf[0][j].x)[d] = o[j];
            }
        }
        if (s == steps - 1) {   // the piece that reaches back over counted entries
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t m = keep_mask(4 * d, skip);
#pragma unroll
                for (int i = 0; i < MT; ++i) (&af[i].x)[d] &= m;
#pragma unroll
                for (int h = 0; h < PL; ++h)
#pragma unroll
                    for (int j = 0; j < 4; ++j) (&bf[h][j].x)[d] &= m;
            }
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) {
#pragma unroll
            for (int i = 0; i < MT; ++i) sa[i] = dot4_ones((&af[i].x)[d], sa[i]);
#pragma unroll
            for (int h = 0; h < PL; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) sb[h][j] = dot4_ones((&bf[h][j].x)[d], sb[h][j]);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int h = 0; h < PL; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[h][i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                        (v4i){(int)af[i].x, (int)af[i].y, (int)af[i].z, (int)af[i].w},
                        (v4i){(int)bf[h][j].x, (int)bf[h][j].y, (int)bf[h][j].z, (int)bf[h][j].w}, acc[h][i][j], 0, 0, 0);
    }
    // byte sums of the tile's rows and columns (index inside an MFMA tile, tile)
#pragma unroll
    for (int i = 0; i < MT; ++i) atomicAdd(&s_rs[sub][i * 16 + l16], sa[i]);
#pragma unroll
    for (int h = 0; h < PL; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) atomicAdd(&s_cs[sub][h][j * 16 + l16], sb[h][j]);

    const Zero z = zero_points(p);
    const bool col_ok = n0 + 4 * l16 < p.cols;
    // results of unit u = (i, r): row idx 4*kb + r of MFMA row tile i, the lane's four columns
    auto row_of = [&](int i, int r, bool &ok) {
        const int idx = kb * 4 + r;
        if (RSA) {
            ok = m0 + 4 * idx < p.rows;
            return min(m0 + 4 * idx, p.rows - 4) + i;
        }
        ok = m0 + i * 16 + idx < p.rows;
        return m0 + i * 16 + idx;
    };
    if (KS == 1) {
        __syncthreads();
        int cs[4], cs1[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            cs[j] = s_cs[sub][0][j * 16 + l16];
            cs1[j] = s_cs[sub][PL - 1][j * 16 + l16];
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                bool ok;
                const int row = row_of(i, r, ok);
                int hi[4], lo[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    hi[j] = acc[0][i][j][r];
                    lo[j] = acc[PL - 1][i][j][r];
                }
                if (ok && col_ok) finish4<WHICH>(p, z, red, row, col0, hi, lo, s_rs[sub][i * 16 + kb * 4 + r], cs, cs1);
            }
    } else {
        // every wavefront leaves its partial tile in LDS and folds its share of the units
        constexpr int SHARE = UNITS / KS;
        int sum[PL][SHARE][4];
#pragma unroll
        for (int h = 0; h < PL; ++h) {
            if (h) __syncthreads();
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *reinterpret_cast<int4 *>(&s_acc[((wave * UNITS + i * 4 + r) * 64 + lane) * 4]) =
                        make_int4(acc[h][i][0][r], acc[h][i][1][r], acc[h][i][2][r], acc[h][i][3][r]);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < SHARE; ++u) {
                int4 t = make_int4(0, 0, 0, 0);
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const int4 v = *reinterpret_cast<const int4 *>(&s_acc[(((sub * KS + k) * UNITS + ks * SHARE + u) * 64 + lane) * 4]);
                    t.x += v.x;
                    t.y += v.y;
                    t.z += v.z;
                    t.w += v.w;
                }
                sum[h][u][0] = t.x;
                sum[h][u][1] = t.y;
                sum[h][u][2] = t.z;
                sum[h][u][3] = t.w;
            }
        }
        int cs[4], cs1[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            cs[j] = s_cs[sub][0][j * 16 + l16];
            cs1[j] = s_cs[sub][PL - 1][j * 16 + l16];
        }
#pragma unroll
        for (int u = 0; u < SHARE; ++u) {
            const int unit = ks * SHARE + u, i = unit >> 2, r = unit & 3;
            bool ok;
            const int row = row_of(i, r, ok);
            if (ok && col_ok) finish4<WHICH>(p, z, red, row, col0, sum[0][u], sum[PL - 1][u], s_rs[sub][i * 16 + kb * 4 + r], cs, cs1);
        }
    }
}

// adds up the slices of a split reduction: 32 neighbouring results per workgroup, eight threads share the slices of a
// result.  Few results and up to 64 slices: the loads of a thread have to be in flight together.
constexpr int kFoldResults = 32, kFoldGroups = 8;
template <bool WIDE>   // int64 results (wgrad)
__global__ __launch_bounds__(kFoldResults * kFoldGroups) void fc_fold(const int64_t *__restrict__ partial, int slices, int64_t count,
                                                                     const q8t_qparams *__restrict__ qa,
                                                                     const q8t_qparams *__restrict__ qb, float *__restrict__ out,
                                                                     void *__restrict__ acc)
{
    __shared__ int64_t part[kFoldGroups][kFoldResults];
    const int e = threadIdx.x % kFoldResults, g = threadIdx.x / kFoldResults;
    const int64_t i = (int64_t)blockIdx.x * kFoldResults + e;
    const float sc = qa->scale * qb->scale;
    int64_t v = 0;
    if (i < count) {
#pragma unroll 8
        for (int z = g; z < slices; z += kFoldGroups) v += partial[z * count + i];
    }
    part[g][e] = v;
    __syncthreads();
    if (g != 0 || i >= count) return;
#pragma unroll
    for (int k = 1; k < kFoldGroups; ++k) v += part[k][e];
    if (WIDE) {
        if (acc) ((int64_t *)acc)[i] = v;
        if (out) out[i] = (float)((double)v * (double)sc);
    } else {
        if (acc) ((int32_t *)acc)[i] = (int32_t)v;
        if (out) out[i] = sc * (float)(int32_t)v;
    }
}

// ---- large products: 128x128 tiles through LDS --------------------------------------------------------------------
constexpr int BM = 128, BN = 128, TT = 256;

// A staged operand of 128 rows (its rows or columns) x 64 reduction indices.  LDS row of (group c of four, member j):
// (c / 16) * 64 + j * 16 + c % 16, so that MFMA tile j of a 64-row block holds the j-th members of 16 groups.
__device__ __forceinline__ int lds_row_member(int lr) { return ((lr >> 6) * 16 + (lr & 15)) * 4 + ((lr >> 4) & 3); }

template <int KIND>   // 0: RF int8, 1: RS int8, 2: RS int16 (two planes)
struct Stage;

template <>
struct Stage<0> {
    const int8_t *p0, *p1;
    uint4 v[2][2];   // [register set][row]
    int s[2];
    int q;
    // grouped: the columns of dgrad, whose LDS rows follow the member order; plain: the rows of A
    __device__ __forceinline__ void init(const void *base, int ld, int first, int count, bool grouped)
    {
        const int ar = threadIdx.x >> 2;
        q = threadIdx.x & 3;
        int r0 = first + ar, r1 = first + ar + 64;
        if (grouped) {
            const int g0 = lds_row_member(ar), g1 = lds_row_member(ar + 64);
            r0 = min(first + (g0 & ~3), count - 4) + (g0 & 3);
            r1 = min(first + (g1 & ~3), count - 4) + (g1 & 3);
        } else {
            r0 = min(r0, count - 1);
            r1 = min(r1, count - 1);
        }
        p0 = (const int8_t *)base + (int64_t)r0 * ld + q * 16;
        p1 = (const int8_t *)base + (int64_t)r1 * ld + q * 16;
        s[0] = s[1] = 0;
    }
    template <int SET>
    __device__ __forceinline__ void load(int k0)
    {
        v[SET][0] = ld16(p0 + k0);
        v[SET][1] = ld16(p1 + k0);
    }
    template <int SET>
    __device__ __forceinline__ void store(int8_t *lds, int skip)
    {
        const int ar = threadIdx.x >> 2;
        uint4 t[2] = {v[SET][0], v[SET][1]};
        if (skip > 0) {
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t m = keep_mask(q * 16 + 4 * d, skip);
                (&t[0].x)[d] &= m;
                (&t[1].x)[d] &= m;
            }
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            s[0] = dot4_ones((&t[0].x)[d], s[0]);
            s[1] = dot4_ones((&t[1].x)[d], s[1]);
        }
        int8_t *o = lds + ar * 64 + ((q ^ swz(ar)) * 16);
        *reinterpret_cast<uint4 *>(o) = t[0];
        *reinterpret_cast<uint4 *>(o + 64 * 64) = t[1];
    }
    __device__ __forceinline__ void sums(int *out)
    {
        const int ar = threadIdx.x >> 2;
        atomicAdd(&out[ar], s[0]);
        atomicAdd(&out[ar + 64], s[1]);
    }
};

// a thread holds 8 reduction indices of one group of four columns
template <>
struct Stage<1> {
    const int8_t *base;
    int ld;
    uint32_t voff;
    uint32_t v[2][8];
    int s[4];
    __device__ __forceinline__ void init(const void *b, int ld_, int first, int count, bool)
    {
        base = (const int8_t *)b;
        ld = ld_;
        const int c = threadIdx.x & 31, k8 = threadIdx.x >> 5;
        voff = (uint32_t)(min(first + 4 * c, count - 4)) + (uint32_t)(k8 * 8) * (uint32_t)ld;
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = 0;
    }
    template <int SET>
    __device__ __forceinline__ void load(int k0)
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[SET][i] = ld4(base + (int64_t)(k0 + i) * ld + voff);
    }
    __device__ __forceinline__ static void put(int8_t *lds, int c, int k8, int j, uint32_t lo, uint32_t hi)
    {
        const int r = (c >> 4) * 64 + j * 16 + (c & 15);
        *reinterpret_cast<uint2 *>(lds + r * 64 + (((k8 >> 1) ^ swz(r)) * 16) + (k8 & 1) * 8) = make_uint2(lo, hi);
    }
    template <int SET>
    __device__ __forceinline__ void store(int8_t *lds, int skip)
    {
        const int c = threadIdx.x & 31, k8 = threadIdx.x >> 5;
        uint32_t a[4], b[4];
        transpose4x4(v[SET][0], v[SET][1], v[SET][2], v[SET][3], a);
        transpose4x4(v[SET][4], v[SET][5], v[SET][6], v[SET][7], b);
        if (skip > 0) {
            const uint32_t ma = keep_mask(k8 * 8, skip), mb = keep_mask(k8 * 8 + 4, skip);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[j] &= ma;
                b[j] &= mb;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s[j] = dot4_ones(a[j], dot4_ones(b[j], s[j]));
            put(lds, c, k8, j, a[j], b[j]);
        }
    }
    __device__ __forceinline__ void sums(int *out)
    {
        const int c = threadIdx.x & 31;
#pragma unroll
        for (int j = 0; j < 4; ++j) atomicAdd(&out[(c >> 4) * 64 + j * 16 + (c & 15)], s[j]);
    }
};

template <>
struct Stage<2> {
    const int16_t *base;
    int ld;
    uint32_t voff;   // elements
    uint2 v[2][8];
    int s[2][4];
    __device__ __forceinline__ void init(const void *b, int ld_, int first, int count, bool)
    {
        base = (const int16_t *)b;
        ld = ld_;
        const int c = threadIdx.x & 31, k8 = threadIdx.x >> 5;
        voff = (uint32_t)(min(first + 4 * c, count - 4)) + (uint32_t)(k8 * 8) * (uint32_t)ld;
#pragma unroll
        for (int j = 0; j < 4; ++j) s[0][j] = s[1][j] = 0;
    }
    template <int SET>
    __device__ __forceinline__ void load(int k0)
    {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[SET][i] = ld8(base + (int64_t)(k0 + i) * ld + voff);
    }
    template <int SET>
    __device__ __forceinline__ void store(int8_t *lds, int skip)
    {
        const int c = threadIdx.x & 31, k8 = threadIdx.x >> 5;
        const uint32_t ma = keep_mask(k8 * 8, skip), mb = keep_mask(k8 * 8 + 4, skip);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t t[8], a[4], b[4];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = h ? lo_bytes(v[SET][i]) : hi_bytes(v[SET][i]);
            transpose4x4(t[0], t[1], t[2], t[3], a);
            transpose4x4(t[4], t[5], t[6], t[7], b);
            if (skip > 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    a[j] &= ma;
                    b[j] &= mb;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                s[h][j] = dot4_ones(a[j], dot4_ones(b[j], s[h][j]));
                Stage<1>::put(lds + h * BN * 64, c, k8, j, a[j], b[j]);
            }
        }
    }
    __device__ __forceinline__ void sums(int *out)
    {
        const int c = threadIdx.x & 31;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) atomicAdd(&out[h * BN + (c >> 4) * 64 + j * 16 + (c & 15)], s[h][j]);
    }
};

template <int WHICH>
__global__ __launch_bounds__(TT, 2) void fc_tile(const FcArgs p)
{
    constexpr int PL = WHICH == WGRAD ? 2 : 1;
    constexpr int KA = WHICH == WGRAD ? 1 : 0, KB = WHICH == FWD ? 1 : (WHICH == DGRAD ? 0 : 2);
    constexpr int A_BYTES = BM * 64, B_BYTES = PL * BN * 64;
    __shared__ __attribute__((aligned(16))) int8_t sA[2 * A_BYTES], sB[2 * B_BYTES];
    __shared__ int s_rs[BM], s_cs[PL * BN];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kb = lane >> 4;
    const int lg = q8t_gemm::xcd_logical(blockIdx.x, p.tiles);
    if (lg >= p.tiles) return;
    // tiles in blocks of 8 rows of tiles: the tiles an XCD works on at a time share both operands
    const int tm = p.tiles / p.tn, per = 8 * p.tn, blk = lg / per, in = lg - blk * per;
    const int bh = min(8, tm - blk * 8);
    const int m0 = (blk * 8 + in % bh) * BM, n0 = (in / bh) * BN;
    for (int i = tid; i < BM; i += TT) s_rs[i] = 0;
    for (int i = tid; i < PL * BN; i += TT) s_cs[i] = 0;

    Stage<KA> sta;
    Stage<KB> stb;
    sta.init(p.a, p.lda, m0, p.rows, false);
    stb.init(p.b, p.ldb, n0, p.cols, true);

    v4i acc[PL][4][4];
#pragma unroll
    for (int h = 0; h < PL; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[h][i][j] = (v4i){0, 0, 0, 0};

    const int steps = (p.red + 63) >> 6;
    const int last0 = p.red - 64, over = steps * 64 - p.red;   // the last step reaches back over `over` counted entries
    auto k0_of = [&](int s) { return min(s * 64, last0); };
    auto skip_of = [&](int s) { return s < steps - 1 ? 0 : (s == steps - 1 ? over : 64); };
    const int ra = (wave & 1) * 64, rb = (wave >> 1) * 64;

#define Q8T_FC_STEP(SET, S)                                                                                     \
    {                                                                                                           \
        const int8_t *a_ = sA + ((S)&1) * A_BYTES, *b_ = sB + ((S)&1) * B_BYTES;                                \
        v4i af[4];                                                                                              \
        _Pragma("unroll") for (int i = 0; i < 4; ++i)                                                           \
        {                                                                                                       \
            const int r = ra + i * 16 + l16;                                                                    \
            af[i] = *reinterpret_cast<const v4i *>(a_ + r * 64 + ((kb ^ swz(r)) * 16));                         \
        }                                                                                                       \
        _Pragma("unroll") for (int h = 0; h < PL; ++h) _Pragma("unroll") for (int j = 0; j < 4; ++j)            \
        {                                                                                                       \
            const int r = rb + j * 16 + l16;                                                                    \
            const v4i bf = *reinterpret_cast<const v4i *>(b_ + h * BN * 64 + r * 64 + ((kb ^ swz(r)) * 16));    \
            _Pragma("unroll") for (int i = 0; i < 4; ++i) acc[h][i][j] =                                        \
                __builtin_amdgcn_mfma_i32_16x16x64_i8(af[i], bf, acc[h][i][j], 0, 0, 0);                        \
        }                                                                                                       \
        sta.template store<SET>(sA + (((S) + 1) & 1) * A_BYTES, skip_of((S) + 1));                              \
        stb.template store<SET>(sB + (((S) + 1) & 1) * B_BYTES, skip_of((S) + 1));                              \
        sta.template load<SET>(k0_of((S) + 3));                                                                 \
        stb.template load<SET>(k0_of((S) + 3));                                                                 \
        q8t_lds_barrier();                                                                                      \
    }
    sta.template load<0>(k0_of(0));
    stb.template load<0>(k0_of(0));
    sta.template load<1>(k0_of(1));
    stb.template load<1>(k0_of(1));
    sta.template store<0>(sA, skip_of(0));
    stb.template store<0>(sB, skip_of(0));
    sta.template load<0>(k0_of(2));
    stb.template load<0>(k0_of(2));
    __syncthreads();
    for (int s = 0; s < steps; s += 2) {
        Q8T_FC_STEP(1, s)
        Q8T_FC_STEP(0, s + 1)   // surplus step: staged zeros
    }
#undef Q8T_FC_STEP
    sta.sums(s_rs);
    stb.sums(s_cs);
    __syncthreads();

    const Zero z = zero_points(p);
    const int cg = n0 + rb + 4 * l16;   // the lane's four columns: member order undone
    const bool col_ok = cg < p.cols;
    const int col0 = min(cg, p.cols - 4);
    int cs[4], cs1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        cs[j] = s_cs[rb + j * 16 + l16];
        cs1[j] = s_cs[(PL - 1) * BN + rb + j * 16 + l16];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int idx = kb * 4 + r, lr = ra + i * 16 + idx;
            int row = m0 + lr;
            bool ok = row < p.rows;
            if (KA == 1) {
                const int g = m0 + ra + 4 * idx;
                ok = g < p.rows;
                row = min(g, p.rows - 4) + i;
            }
            int hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                hi[j] = acc[0][i][j][r];
                lo[j] = acc[PL - 1][i][j][r];
            }
            if (ok && col_ok) finish4<WHICH>(p, z, p.red, row, col0, hi, lo, s_rs[lr], cs, cs1);
        }
}

// ---- large products of aligned matrices: tiles that go to LDS without registers -----------------------------------
// 128 rows x 128 byte columns a workgroup (weight gradient: 64 columns, the two bytes of a 16-bit code are neighbouring byte
// columns), K-steps of 128 in two LDS buffers.  A tile of either operand is 128 LDS rows of 128 bytes, eight 16-byte pieces
// each, which global_load_lds writes as 64 lanes x 16 bytes in a row; so the permutation that keeps the fragment reads free
// of bank conflicts is applied to the addresses in memory: piece s of LDS row r holds the operand's piece s ^ perm(r).
//   RF operand: LDS row = row of the operand, pieces along the reduction; a fragment is one ds_read_b128
//   RS operand: LDS row = reduction index, pieces along the columns; a fragment is two ds_read_b64_tr_b8, in which 16 lanes
//               read 8 rows x 16 bytes and lane i receives the 8 bytes of column i
// Nothing is transposed or split on the way.  2048x4096x4096, us, against fc_tile: forward 69 / 45, layer gradient 60 / 46, weight
// gradient 111 / 101; 2048^3 31 / 19, 26 / 19, 43 / 31; matrix units 42, 43 and 40% busy (fc_tile 20, 23, 26).  Whole lines (K-steps of 128: of 64 the
// same loop takes 47 us for 37 here), no registers between memory and LDS and the second workgroup of a compute unit are what
// it lives on: tiles of 128x256 and three or four buffers, one workgroup a unit, take as long; 32x32x32 products are slower (43).
constexpr int DT = 512, DK = 128, DTILE = 128 * DK;   // threads, reduction indices a step, bytes of an operand's tile

__device__ __constant__ __align__(16) int8_t fc_zeros[16] = {};   // what pieces outside an operand read

// One operand's share of the staging: two pieces per thread and step.
template <bool RS>
struct DmaStage {
    const int8_t *src[2];
    size_t step[2];      // bytes from step to step
    int at[2];           // reduction index of the piece in step 0
    __device__ __forceinline__ static int perm(int r)
    {
        // RS: eight neighbouring reduction indices on four pieces, indices 16 apart on others
        return RS ? ((r >> 1) & 3) | ((r >> 2) & 4) : (r >> 1) & 7;
    }
    // first / count: rows (RF) or byte columns (RS) of the operand; ld in bytes
    __device__ __forceinline__ void init(const void *base, int64_t ld, int first, int count)
    {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int p = u * DT + (int)threadIdx.x, r = p >> 3, q = (p & 7) ^ perm(r);
            if (RS) {
                const bool in = first + q * 16 < count;   // the columns of the piece exist
                at[u] = r;
                src[u] = in ? (const int8_t *)base + r * ld + first + q * 16 : fc_zeros;
                step[u] = in ? (size_t)DK * ld : 0;
            } else {
                at[u] = q * 16;
                src[u] = (const int8_t *)base + min(first + r, count - 1) * ld + q * 16;
                step[u] = DK;
            }
        }
    }
    // left: reduction indices from this step on
    __device__ __forceinline__ void issue(int8_t *lds, int left)
    {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int8_t *g = src[u];
            if (left < DK && at[u] >= left) g = fc_zeros;
            q8t_gemm::copy16_to_lds(g, lds + (u * DT + wave * 64) * 16);
            src[u] += step[u];
        }
    }
    // the 16 reduction indices h * 64 + 16 * kb .. of row / byte column `c16` * 16 + l16
    __device__ __forceinline__ static v4i fragment(const int8_t *lds, int c16, int h, int l16, int kb)
    {
        if (!RS) {
            const int r = c16 * 16 + l16;
            return *reinterpret_cast<const v4i *>(lds + r * DK + (((h * 4 + kb) ^ perm(r)) * 16));
        }
        typedef int v2i __attribute__((ext_vector_type(2)));
        v2i t[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int k = h * 64 + kb * 16 + e * 8 + (l16 >> 1);
            const int8_t *a = lds + k * DK + ((c16 ^ perm(k)) * 16) + (l16 & 1) * 8;
            t[e] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i *)(int8_t *)a);
        }
        return (v4i){t[0][0], t[0][1], t[1][0], t[1][1]};
    }
};

template <int WHICH>
__global__ __launch_bounds__(DT, 4) void fc_dma(const FcArgs p)
{
    constexpr bool RSA = WHICH == WGRAD, RSB = WHICH != DGRAD;
    constexpr int WR = 2, WC = 4, MT = 4, NT = 2;   // wavefronts down and across, 16x16 tiles of a wavefront
    constexpr int CB = WHICH == WGRAD ? 2 : 1;      // byte columns per column
    constexpr int COLS = 128 / CB, STAGE = 2 * DTILE;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];   // two buffers of A and B tiles

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kb = lane >> 4;
    const int lg = q8t_gemm::xcd_logical(blockIdx.x, p.tiles);
    if (lg >= p.tiles) return;
    // tiles in blocks of 8 rows of tiles: the tiles an XCD works on at a time share both operands
    const int tm = p.tiles / p.tn, per = 8 * p.tn, blk = lg / per, in = lg - blk * per;
    const int bh = min(8, tm - blk * 8);
    const int m0 = (blk * 8 + in % bh) * 128, n0 = (in / bh) * COLS;   // rows, columns
    const int wr = wave % WR, wc = wave / WR;

    DmaStage<RSA> sta;
    DmaStage<RSB> stb;
    sta.init(p.a, p.lda, m0, p.rows);
    stb.init(p.b, (int64_t)p.ldb * CB, n0 * CB, p.cols * CB);
    auto issue = [&](int s, int8_t *to) {
        sta.issue(to, p.red - s * DK);
        stb.issue(to + DTILE, p.red - s * DK);
    };

    v4i acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (v4i){0, 0, 0, 0};
    // Byte sums, as products with ones (forward, us: without sums 43, as v_dot4 on the fragments 48 to 51, so 46): the
    // wavefronts that share rows (columns) take a row tile (column tile) each, the first one they multiply: a wavefront goes
    // round its tiles from there.
    static_assert(MT == WC && NT == WR, "a tile per wavefront");
    const v4i ones = (v4i){0x01010101, 0x01010101, 0x01010101, 0x01010101};
    v4i rsum = (v4i){0, 0, 0, 0}, csum = (v4i){0, 0, 0, 0};
    auto row_tile = [&](int i) { return wr * MT + ((i + wc) & (MT - 1)); };
    auto col_tile = [&](int j) { return wc * NT + ((j + wr) & (NT - 1)); };
    const uint32_t flip = WHICH == WGRAD && !(l16 & 1) ? 0x80808080u : 0u;   // low bytes are re-centred

    const int steps = (p.red + DK - 1) / DK;
    issue(0, smem);
    v4i af[2][MT], bf[2][NT];
    auto read = [&](const int8_t *a, int h) {
#pragma unroll
        for (int j = 0; j < NT; ++j) bf[h][j] = DmaStage<RSB>::fragment(a + DTILE, col_tile(j), h, l16, kb);
#pragma unroll
        for (int i = 0; i < MT; ++i) af[h][i] = DmaStage<RSA>::fragment(a, row_tile(i), h, l16, kb);
    };
    auto multiply = [&](int h) {
        if (WHICH == WGRAD) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int d = 0; d < 4; ++d) bf[h][j][d] ^= (int)flip;
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[h][i], bf[h][j], acc[i][j], 0, 0, 0);
        rsum = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[h][0], ones, rsum, 0, 0, 0);
        csum = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, bf[h][0], csum, 0, 0, 0);
    };
    auto step = [&](int s, const int8_t *cur, int8_t *nxt) {
        // the tiles of this step are there, and every wavefront is past its reads of the other buffer
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (s + 1 < steps) issue(s + 1, nxt);
        read(cur, 0);
        read(cur, 1);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);   // a wavefront that multiplies goes before the ones that read (46 -> 45 us)
        multiply(0);
        multiply(1);
        __builtin_amdgcn_s_setprio(0);
    };
    for (int s = 0; s < steps; s += 2) {
        step(s, smem, smem + STAGE);
        if (s + 1 < steps) step(s + 1, smem + STAGE, smem);
    }
    __syncthreads();
    int *s_rs = reinterpret_cast<int *>(smem), *s_cs = s_rs + 128;   // [128] each
    if (l16 == 0) *reinterpret_cast<v4i *>(&s_rs[row_tile(0) * 16 + kb * 4]) = rsum;   // every column holds the sums
    // every row does; the zeros behind the reduction went in as low bytes of -128
    if (kb == 0) s_cs[col_tile(0) * 16 + l16] = csum[0] + (flip ? 128 * (steps * DK - p.red) : 0);
    __syncthreads();

    const Zero z = zero_points(p);
    if (WHICH != WGRAD) {
        const uint32_t kzz = (uint32_t)p.red * (uint32_t)z.za * (uint32_t)z.zb;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int lc = col_tile(j) * 16 + l16, col = n0 + lc;
            const uint32_t cs = (uint32_t)z.za * (uint32_t)s_cs[lc];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int lr = row_tile(i) * 16 + kb * 4 + r, row = m0 + lr;
                    const int c = (int)((uint32_t)acc[i][j][r] + kzz - (uint32_t)z.zb * (uint32_t)s_rs[lr] - cs);   // fits by contract
                    if (row < p.rows && col < p.cols) {
                        const int64_t o = (int64_t)row * p.cols + col;
                        if (p.acc) ((int32_t *)p.acc)[o] = c;
                        if (p.out) p.out[o] = z.sc * (float)c;
                    }
                }
        }
    } else {
        // a lane pair holds the low and the high byte products of a column: the even lane finishes rows 0, 1 of the four, the
        // odd one rows 2, 3; results go through LDS so that they leave in whole lines
        // The sums are integers below 2^53 in magnitude (65536 products of 255 * 65535): in double they and the correction are exact
        // and take a fifth of the instructions of 64-bit integers (16.8 M results: 20 us of vector instructions before).
        constexpr int TP = COLS + 4;
        float *turn = reinterpret_cast<float *>(smem + 4096);            // [128][TP]
        double *s_t = reinterpret_cast<double *>(smem + 2048);           // the rows' share of the correction
        if (tid < 128)
            s_t[tid] = (double)(128 - z.zb) * (double)s_rs[tid] + (double)p.red * (double)z.za * (double)(z.zb - 128);
        __syncthreads();
        const bool odd = l16 & 1;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int lb = col_tile(j) * 16 + l16, lc = lb >> 1, col = n0 + lc;
            const double cs = (double)z.za * (256.0 * (double)s_cs[lb | 1] + (double)s_cs[lb & ~1]);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                int other[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) other[r] = __builtin_amdgcn_mov_dpp(acc[i][j][r], 0xB1, 0xF, 0xF, true);   // lane ^ 1
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int hi = odd ? acc[i][j][2 + k] : other[k], lo = odd ? other[2 + k] : acc[i][j][k];
                    const int lr = row_tile(i) * 16 + kb * 4 + (odd ? 2 : 0) + k, row = m0 + lr;
                    const double c = (256.0 * (double)hi + (double)lo) + (s_t[lr] - cs);
                    turn[lr * TP + lc] = (float)(c * (double)z.sc);
                    if (p.acc && row < p.rows && col < p.cols) ((int64_t *)p.acc)[(int64_t)row * p.cols + col] = (int64_t)c;
                }
            }
        }
        __syncthreads();
        if (p.out) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = u * DT + tid, lr = e / (COLS / 4), lc = e % (COLS / 4) * 4, row = m0 + lr, col = n0 + lc;   // cols is a multiple of 8
                if (row < p.rows && col < p.cols) {
                    const float4 v = *reinterpret_cast<const float4 *>(&turn[lr * TP + lc]);
                    float *d = p.out + (int64_t)row * p.cols + col;
                    if (p.vec) {
                        *reinterpret_cast<float4 *>(d) = v;
                    } else {
                        d[0] = v.x;
                        d[1] = v.y;
                        d[2] = v.z;
                        d[3] = v.w;
                    }
                }
            }
        }
    }
}

constexpr int kMaxRed = 65536;   // |a*b| <= 2^14 per product of two signed bytes: partial sums stay below 2^31

struct Plan {
    int rows, cols, red;
    int tile;               // fc_tile instead of fc_direct
    int tn;                 // column tiles
    int64_t tiles;
    int ks, slice, slices;  // fc_direct: wavefronts per tile, K-steps per slice of the reduction, slices
};

Plan plan_for(int which, int M, int N, int K)
{
    Plan p;
    p.rows = which == 2 ? K : M;
    p.cols = which == 1 ? K : N;
    p.red = which == 0 ? K : (which == 1 ? N : M);
    const int64_t t128 = (int64_t)((p.rows + 127) / 128) * ((p.cols + 127) / 128);
    const int steps = (p.red + 63) / 64;
    p.ks = p.slices = 1;
    p.slice = steps;
    // 128x128 tiles from half a tile per compute unit on (tiles / fc_direct, us): 1500x1500x1500, 144 tiles, 22.6 / 22.1 forward,
    // 18.5 / 20.2 dgrad; 2048x1024 results, 128 tiles, over 2048: 25.7 / 20.7, 20.5 / 26.6; the forward of 2048x616x3680, 80
    // tiles, 39.7 / 30.1.  The weight gradient's fc_direct holds 64 KB of LDS per tile of 64x64, so 512 of those, 128 of these,
    // are one round of workgroups and more are two: 128 tiles over 128 and 2048 10.9 / 12.2 and 39.2 / 29.0, 144 11.1 / 17.3 and
    // 39.4 / 41.8.  With a single K-step a result narrower than a tile pays for the padding (weight gradient 65536x16x64 13.5
    // against 8.6).
    p.tile = t128 >= (which == 2 ? 140 : 128) && (p.red > 64 || (p.red == 64 && p.rows > 64 && p.cols > 64));
    p.tn = p.tile ? (p.cols + 127) / 128 : (p.cols + 63) / 64;
    const int tr = which == 2 ? 64 : 32;
    p.tiles = p.tile ? t128 : (int64_t)((p.rows + tr - 1) / tr) * p.tn;
    if (p.tile) return p;
    // wavefronts per tile: enough of them to fill the chip (two per SIMD; limits of 512 .. 8192 wavefronts were swept, and
    // fewer leave the 512x2048x2048 forward at 24 instead of 10.5 us), no more than there are K-steps
    while (p.ks < 8 && 2 * p.ks <= steps && p.tiles * p.ks < 2048) p.ks *= 2;
    // A tile is shared by four wavefronts even where they outnumber the K-steps: they share its results, too (64-bit
    // arithmetic in the weight gradient).  One K-step, 64x64x256: 4.9 / 5.2 / 8.4 -> 3.8 / 3.8 / 6.1 us; with 460 tiles
    // the weight gradient is back to 8.6 with a wavefront a tile against 10.9.
    if (p.ks == 2 || (p.ks == 1 && p.tiles <= 256)) p.ks = 4;
    // Few tiles: slices of the reduction, two K-steps per wavefront or more, as many as give every compute unit a
    // workgroup.  Unsplit -> split: weight gradient 16x16x65536 198 -> 11 us, 64x64x4096 18.1 -> 10.8, 12x237x2065 14.2 ->
    // 12.1, 1000x256x4096 (64 tiles) 19.6 -> 18.3; forward 64x64x16384 24.4 -> 7.0, 64x64x4096 8.7 -> 6.7; layer gradient
    // 16x64x4096 12.0 -> 7.2.  Two or three slices over more tiles cost what they gain until the reduction is longer (128
    // tiles: 64 K-steps 9.5 -> 13.3, 79 30.6 -> 21.9).
    if (p.ks == 8 && steps >= 32 && (p.tiles <= 64 || steps >= 128)) {
        const int n = min((int)min((int64_t)64, 256 / p.tiles), steps / 16);
        if (n > 1) {
            p.slice = (steps + n - 1) / n;
            p.slices = (steps + p.slice - 1) / p.slice;
        }
    }
    return p;
}

// fc_dma: 16-byte pieces that lie whole inside or outside of the operands, at 16-byte addresses, and tiles for half the compute
// units.  us, fc_dma / the kernel that plan_for names: forward, 104 tiles over 2816 21.4 / 28.8, 114 over 576 10.5 / 10.9, 80 over
// 2528 19.8 / 24.2, 68 over 3248 27.9 / 29.0, 90 over 128 7.9 / 7.3, 63 over 544 9.9 / 7.2; layer gradient 96 over 688 10.9 / 10.3, 100
// over 1936 17.3 / 20.1; weight gradient (tiles of 64 columns) 130 over 1584 15.8 / 24.8.  The weight gradient's fc_direct runs a round of 256
// tiles of 64x64 at once and shares their reduction among wavefronts, so up to there it stays: results of 256x4096 over 65536 (128
// tiles) 534 / 311, 1024x1024 over 4096 28 / 23; 447 sizes: 0.2% slower than the better of the two, 0.5 with a line at 112 tiles.
// Results narrower than three quarters of a tile stay away: they would multiply zeros.
bool dma_wanted(int which, const FcArgs &p)
{
    const int bytes = which == 2 ? 2 : 1, cols = 128 / bytes;
    if (!(q8t_aligned(p.a, 16) && q8t_aligned(p.b, 16) && p.lda % 16 == 0 && p.ldb * bytes % 16 == 0)) return false;
    if (p.red < 64 || p.rows < 96 || p.cols < cols * 3 / 4) return false;
    const int64_t tiles = (int64_t)((p.rows + 127) / 128) * ((p.cols + cols - 1) / cols);   // below 2^20: a matrix has fewer than 2^31 entries
    return which == 2 ? (int64_t)((p.rows + 63) / 64) * ((p.cols + 63) / 64) > 256 : tiles >= 128 || (tiles >= 80 && p.red >= 1024);
}

}  // namespace

// sizes the kernels above take: whole groups of four columns (rows) and one 16-entry piece of the reduction exist
bool q8t_fc_supported(int which, int M, int N, int K)
{
    // A reduction of less than one K-step under many results is bound by their stores.  Up to about the size of the last
    // cache the general kernel's leave faster (16384x1000x16 25 against 30 us, 65536x1000x16 79 against 104), beyond it not
    // (16384x16384x16 401 against 340), and below 4 M results neither (2280x1571x18 10.8 both).
    const int64_t results = (int64_t)M * (which == 0 ? N : K);
    if (which < 2 && (which == 0 ? K : N) < 64 && results >= 4000000 && results <= (1 << 27)) return false;
    if (which == 0) return K >= 16 && N >= 4;
    if (which == 1) return N >= 16 && K >= 4;
    return M >= 16 && M <= kMaxRed && N >= 4 && K >= 4;
}

size_t q8t_fc_ws(int which, int M, int N, int K)
{
    const Plan pl = plan_for(which, M, N, K);
    return pl.slices > 1 ? (size_t)pl.slices * pl.rows * pl.cols * sizeof(int64_t) : 0;
}

int q8t_fc(int which, const void *a, const q8t_qparams *qa, const void *b, const q8t_qparams *qb, int M, int N, int K,
           float *out_f, void *out_acc, void *ws, hipStream_t st)
{
    const Plan pl = plan_for(which, M, N, K);
    if (pl.slices > 1 && (!ws || !q8t_aligned(ws, 8))) return Q8T_ERR_WORKSPACE;
    FcArgs p;
    p.a = (const int8_t *)a;
    p.b = b;
    p.qa = qa;
    p.qb = qb;
    p.rows = pl.rows;
    p.cols = pl.cols;
    p.red = pl.red;
    p.lda = which == 1 ? N : K;
    p.ldb = N;
    p.out = out_f;
    p.acc = out_acc;
    p.partial = pl.slices > 1 ? (int64_t *)ws : nullptr;
    p.slice = pl.slice;
    p.vec = p.cols % 4 == 0 && q8t_aligned(out_f, 16);
    p.tn = pl.tn;
    p.tiles = (int)pl.tiles;
    if (dma_wanted(which, p)) {
        const int cols = which == 2 ? 64 : 128;
        p.tn = (p.cols + cols - 1) / cols;
        p.tiles = (p.rows + 127) / 128 * p.tn;
        const dim3 grid(q8t_gemm::xcd_grid(p.tiles));
        constexpr size_t lds = 4 * DTILE;
        if (which == 0) hipLaunchKernelGGL(fc_dma<FWD>, grid, dim3(DT), lds, st, p);
        else if (which == 1) hipLaunchKernelGGL(fc_dma<DGRAD>, grid, dim3(DT), lds, st, p);
        else hipLaunchKernelGGL(fc_dma<WGRAD>, grid, dim3(DT), lds, st, p);
        Q8T_LAUNCH_CHECK();
        return Q8T_OK;
    }
    if (pl.tile) {
        const dim3 grid(q8t_gemm::xcd_grid(pl.tiles));
        if (which == 0) hipLaunchKernelGGL(fc_tile<FWD>, grid, dim3(TT), 0, st, p);
        else if (which == 1) hipLaunchKernelGGL(fc_tile<DGRAD>, grid, dim3(TT), 0, st, p);
        else hipLaunchKernelGGL(fc_tile<WGRAD>, grid, dim3(TT), 0, st, p);
        Q8T_LAUNCH_CHECK();
        return Q8T_OK;
    }
#define Q8T_GO(W, WAVES, KS)                                                                                                  \
    hipLaunchKernelGGL((fc_direct<W, WAVES, KS>), dim3((unsigned)((pl.tiles + (WAVES / KS) - 1) / (WAVES / KS)), (unsigned)pl.slices), \
                       dim3(WAVES * 64), 0, st, p)
    if (which == 0) { if (pl.ks == 8) Q8T_GO(FWD, 8, 8); else if (pl.ks == 4) Q8T_GO(FWD, 4, 4); else Q8T_GO(FWD, 4, 1); }
    else if (which == 1) { if (pl.ks == 8) Q8T_GO(DGRAD, 8, 8); else if (pl.ks == 4) Q8T_GO(DGRAD, 4, 4); else Q8T_GO(DGRAD, 4, 1); }
    else { if (pl.ks == 8) Q8T_GO(WGRAD, 8, 8); else if (pl.ks == 4) Q8T_GO(WGRAD, 4, 4); else Q8T_GO(WGRAD, 4, 1); }
#undef Q8T_GO
    Q8T_LAUNCH_CHECK();
    if (pl.slices > 1) {
        const int64_t count = (int64_t)pl.rows * pl.cols;
        const dim3 grid((unsigned)((count + kFoldResults - 1) / kFoldResults)), block(kFoldResults * kFoldGroups);
        if (which == 2)
            hipLaunchKernelGGL(fc_fold<true>, grid, block, 0, st, (const int64_t *)ws, pl.slices, count, qa, qb, out_f, out_acc);
        else
            hipLaunchKernelGGL(fc_fold<false>, grid, block, 0, st, (const int64_t *)ws, pl.slices, count, qa, qb, out_f, out_acc);
        Q8T_LAUNCH_CHECK();
    }
    return Q8T_OK;
}
