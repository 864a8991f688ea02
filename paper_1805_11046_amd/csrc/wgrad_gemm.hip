// General MFMA path for the convolution weight gradient g_W = g_l * I^T with the 16-bit copy of
// the gradient (Sections 1 and 4, "gradient bifurcation"): any filter size, stride, padding and
// channel count.  The reduction runs over every output position (n, p, q), which is the
// contiguous index of both NCHW operands, so the product is a GEMM of two matrices that are both
// stored "reduction index fastest":
//
//   A'[2K][Mp]   rows k      : high bytes of the stored 16-bit gradient codes of output channel k
//                rows K + k  : their low bytes, re-centred ( s = 256*hi + lo + 128, hi and lo signed bytes )
//   B'[CRS][Mp]  column (c,r,s) : the input code that meets gradient position m under filter tap (r,s)
//
// Mostly B' is not written: both operands are laid out on padded planes of one pitch, where a tap is an offset into the row of
// its input channel.  Where planes are so small under the filter that this is mostly padding, the input has a plane per tap (B').
//
// Launches: pad_operands or tap_operands (A' and the input), gemm_nt (int8 MFMA, 256x256, 128x128 or 128x64
// tiles, the reduction split into slices of at most 65536 products so that the
// 32-bit accumulators cannot overflow), wgrad_finish (sums the slices in 64 bits, recombines the
// two byte planes, applies the zero-point correction, dequantizes).  Exact for any reduction
// length: every partial sum is an integer below 2^31 and the recombination is done in int64.
// Whole calls, us, against byte planes + im2col rows + a GEMM without shared tiles: 96 -> 200 3x3 @27 batch 50 90 -> 55,
// 64 -> 64 5x5 @56 batch 128 530 -> 208, 48 -> 80 3x3 @32 batch 64 50 -> 40, 112 -> 96 1x1 @56 batch 32 51 -> 34, 208 -> 160
// 3x3/2 @14 batch 64 42 -> 32, 48 -> 64 3x3 @3 batch 300 28 -> 18, 128 -> 128 5x5 @4 batch 100 (49 positions for 16) 31 -> 28.
#include "q8t_common.h"
#include "q8t_internal.h"
#include "gemm_core.h"

namespace {

using q8t_gemm::v4i;

constexpr int kThreads = 256;
constexpr int BM = 128;
constexpr int kMaxSlice = 65536;

__device__ __forceinline__ int bytesum4(uint32_t v) { return __builtin_amdgcn_sdot4((int)v, 0x01010101, 0, false); }
__device__ __forceinline__ int bytesum16(const uint4 &v)
{
    return bytesum4(v.x) + bytesum4(v.y) + bytesum4(v.z) + bytesum4(v.w);
}

// quotient x / d for 0 <= x < 2^24 through the float reciprocal, corrected by at most one
__device__ __forceinline__ int fdiv(int x, int d, float rd)
{
    int q = (int)((float)x * rd);
    const int r = x - q * d;
    if (r < 0) --q;
    else if (r >= d) ++q;
    return q;
}

// ---- operands on padded planes --------------------------------------------------------------------
// The gradient and the input are laid out on planes of the same pitch, so that a filter tap is a constant
// offset into the row of its input channel and all taps of a channel share that row.  With i = r / stride, a = r % stride
// and j = s / stride, b = s % stride, gradient position (p, q) meets plane (a, b) of the input at (p + i, q + j):
//   A'[2K][Mp]            byte planes of the gradient at m = (n*PR + p)*PC + q, both bytes 0 at the pad positions
//   X'[(a, b)][C][XL]     input code at (row*stride + a - pad, col*stride + b - pad) of image n, the zero code outside
//   column (c, r, s)   =  X'[(a, b)][c] + i*PC + j, read as it lies (16-byte loads at any address)
//   mask[Mp]              1 at the real positions: a column's byte sum may count nothing else
// Planes share their pad columns (rows) with the next row (image) as far as both sides are padding.
struct PadG {
    int N, C, H, W, K, P, Q, stride, pad;
    int ra, sa;              // input planes per channel
    int PC, IS;              // row pitch, positions per image
    int64_t Mp, XL;          // lengths of a row of A' and of X'
    int chunks;              // kPadChunk positions each
    int rows, gblocks, xblocks;   // channels per workgroup; blocks of them in the gradient, in one input plane
};
constexpr int kPadChunk = 4 * kThreads;   // positions per workgroup

// A lane owns four positions and walks the channels of its workgroup: where the codes of its positions lie inside an image is
// the same for every channel, so the divisions are paid once and a channel costs a load, two byte permutes (one) and two
// stores (one).  The codes are neighbours in memory except for the pads between them: one load of four codes holds them all,
// unless the group spans two images, the plane is smaller than the load or codes are skipped (stride > 1).
// 96 -> 200 channels @27, batch 50 (18 MB in, 20 MB out): 10 us; byte planes and im2col rows in launches of their own
// (46 MB out) 42.5 us, one channel per workgroup 19 to 24.
__global__ __launch_bounds__(kThreads) void pad_operands(const int16_t *__restrict__ g16, const int8_t *__restrict__ x, PadG g,
                                                         const q8t_qparams *__restrict__ qpx, int8_t *__restrict__ A,
                                                         int8_t *__restrict__ X, int8_t *__restrict__ mask)
{
    int by = blockIdx.y;
    const bool grad = by < g.gblocks;
    by -= grad ? 0 : g.gblocks;
    const int cls = grad ? 0 : by / g.xblocks, a = cls / g.sa, b = cls - a * g.sa;
    const int c0 = (by - cls * g.xblocks) * g.rows, channels = grad ? g.K : g.C, c1 = min(c0 + g.rows, channels);
    const int h0 = grad ? 0 : a - g.pad, w0 = grad ? 0 : b - g.pad, step = grad ? 1 : g.stride;
    const int hend = grad ? g.P : g.H, wend = grad ? g.Q : g.W, plane = hend * wend;
    const uint32_t len = (uint32_t)(grad ? g.Mp : g.XL);
    const int PR = g.IS / g.PC;
    const float rIS = 1.0f / (float)g.IS, rPC = 1.0f / (float)g.PC;
    for (uint32_t chunk = blockIdx.x; chunk < (uint32_t)g.chunks; chunk += gridDim.x) {
        const uint32_t m0 = chunk * kPadChunk, off = threadIdx.x * 4, m = m0 + off;
        if (m >= len) break;
        const uint32_t n_first = m0 / (uint32_t)g.IS;   // uniform
        const int t = (int)(m0 - n_first * (uint32_t)g.IS + off);
        const bool small = g.IS < (1 << 22);            // the quotient by a float reciprocal is exact
        const int dn = small ? fdiv(t, g.IS, rIS) : t / g.IS, rem = t - dn * g.IS;
        int n = (int)n_first + dn, pr = small ? fdiv(rem, g.PC, rPC) : rem / g.PC, pc = rem - pr * g.PC;
        const int n0 = n;
        int place[4], image[4];
        uint32_t real = 0;
        bool one = step == 1 && plane >= 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int h = pr * step + h0, w = pc * step + w0;
            const bool in = n < g.N && (unsigned)h < (unsigned)hend && (unsigned)w < (unsigned)wend;
            place[j] = h * wend + w;
            image[j] = n;
            real |= in ? 1u << j : 0u;
            one = one && (!in || n == n0);
            if (++pc == g.PC) {
                pc = 0;
                if (++pr == PR) {
                    pr = 0;
                    ++n;
                }
            }
        }
        // the load: four codes from `from` on, inside the plane; sel: which of them each position takes, 8: none
        int from = plane - 4;
#pragma unroll
        for (int j = 3; j >= 0; --j)
            if (real >> j & 1) from = min(place[j], plane - 4);
        uint32_t sel[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sel[j] = real >> j & 1 ? (uint32_t)(place[j] - from) : 8u;
            one = one && (sel[j] < 4 || sel[j] == 8);   // a row of positions may be shorter than a row of codes
        }
        const int64_t image_step = (int64_t)channels * plane;
        const int64_t base = real && one ? n0 * image_step + from : 0;
        const uint32_t ones = (real & 1u) | (real & 2u) << 7 | (real & 4u) << 14 | (real & 8u) << 21;
        if (grad) {
            if (by == 0) *reinterpret_cast<uint32_t *>(mask + m) = ones;
            uint32_t shi = 0, slo = 0;   // byte selectors: 2 i + 1 / 2 i of the code's pair, 0x0C: zero
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                shi |= (sel[j] < 8 ? 2 * sel[j] + 1 : 0x0Cu) << (8 * j);
                slo |= (sel[j] < 8 ? 2 * sel[j] : 0x0Cu) << (8 * j);
            }
            const uint32_t flip = ones << 7;
            uint32_t *hi = reinterpret_cast<uint32_t *>(A + (size_t)c0 * g.Mp + m);
            uint32_t *lo = reinterpret_cast<uint32_t *>(A + (size_t)(g.K + c0) * g.Mp + m);
            if (one) {
                const int16_t *src = g16 + base + (int64_t)c0 * plane;
#pragma unroll 4
                for (int c = c0; c < c1; ++c) {
                    uint32_t w[2];
                    __builtin_memcpy(w, src, 8);
                    *hi = __builtin_amdgcn_perm(w[1], w[0], shi);
                    *lo = __builtin_amdgcn_perm(w[1], w[0], slo) ^ flip;
                    src += plane;
                    hi += g.Mp >> 2;
                    lo += g.Mp >> 2;
                }
            } else {
                for (int c = c0; c < c1; ++c) {
                    uint32_t h = 0, l = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (real >> j & 1) {
                            const uint32_t v = (uint16_t)g16[image[j] * image_step + (int64_t)c * plane + place[j]];
                            h |= (v >> 8) << (8 * j);
                            l |= (v & 255u) << (8 * j);
                        }
                    *hi = h;
                    *lo = l ^ flip;
                    hi += g.Mp >> 2;
                    lo += g.Mp >> 2;
                }
            }
        } else {
            const uint32_t zb = (uint32_t)(qpx->zero_point - (1 << (qpx->bits - 1))) & 255u;
            uint32_t s = 0;   // byte selectors: 0..3 the codes, 4 the zero code
#pragma unroll
            for (int j = 0; j < 4; ++j) s |= (sel[j] < 8 ? sel[j] : 4u) << (8 * j);
            uint32_t *dst = reinterpret_cast<uint32_t *>(X + ((size_t)cls * g.C + c0) * g.XL + m);
            if (one) {
                const int8_t *src = x + base + (int64_t)c0 * plane;
#pragma unroll 4
                for (int c = c0; c < c1; ++c) {
                    uint32_t w;
                    __builtin_memcpy(&w, src, 4);
                    *dst = __builtin_amdgcn_perm(zb, w, s);
                    src += plane;
                    dst += g.XL >> 2;
                }
            } else {
#pragma unroll 2
                for (int c = c0; c < c1; ++c) {
                    uint32_t d = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        d |= (real >> j & 1 ? (uint32_t)(uint8_t)x[image[j] * image_step + (int64_t)c * plane + place[j]] : zb) << (8 * j);
                    *dst = d;
                    dst += g.XL >> 2;
                }
            }
        }
    }
}

// Planes of one to three results, a plane of the input per tap: the lanes above would gather their positions from as many
// images, a line of memory for each.  Here a workgroup takes the codes of CG channels of NI images to LDS as they lie and picks the
// rows out of them, four positions a store; a lane's positions are the same in every row.  Images lie an odd number of dwords
// apart, 64 of them a dword further: the lanes of a store, four images apart where a plane has one position, meet
// different banks.  Whole calls, pad_operands / here: 256 -> 512 1x1 over 65536 planes of one position 312 / 120 us, 64 -> 64 3x3/2
// @2 over as many 335 / 60.
struct TapG {
    int NI;              // images of a workgroup
    int CGg, CGx;        // channels of a workgroup, gradient and input
    int pitchg, pitchx;  // bytes from image to image in LDS
    int gblocks, xblocks;
    unsigned gx;
    size_t lds;
};
__host__ __device__ __forceinline__ int tap_image(int i, int pitch) { return i * pitch + (i >> 6) * 4; }

// GRAD: 16-bit codes, every position under one tap, rows of high and of low bytes (0 beyond the last image); else the zero code zb
template <bool GRAD>
__device__ __forceinline__ void tap_rows(int8_t *codes, const int8_t *__restrict__ src, int n0, int ni, int NI, int channels, int c0, int cg,
                                         int H, int W, int P, int Q, int stride, int pad, int S, int taps, int pitch, uint32_t zb,
                                         int8_t *__restrict__ out, int64_t len, int8_t *__restrict__ lo, int8_t *__restrict__ mask)
{
    constexpr int E = GRAD ? 2 : 1;
    const int tid = threadIdx.x, HW = H * W, bytes = cg * HW * E, pieces = (bytes + 15) >> 4;
    for (int i = tid; i < ni * pieces; i += kThreads) {
        const int img = i / pieces, at = (i - img * pieces) * 16;
        const int8_t *a = src + ((int64_t)(n0 + img) * channels + c0) * HW * E + at;
        int8_t *d = codes + tap_image(img, pitch) + at;
        if (at + 16 <= bytes) {
            uint32_t v[4];
            __builtin_memcpy(v, a, 16);
#pragma unroll
            for (int k = 0; k < 4; ++k) reinterpret_cast<uint32_t *>(d)[k] = v[k];
        } else {
            for (int k = 0; k < bytes - at; ++k) d[k] = a[k];
        }
    }
    __syncthreads();
    const int PQ = P * Q, dwords = NI * PQ >> 2, side = kThreads / dwords;   // rows side by side
    const int row0 = tid / dwords, dw = tid - row0 * dwords;
    const int64_t m = (int64_t)n0 * PQ + dw * 4;
    if (row0 >= side || m >= len) return;
    int at[4], h[4], w[4];
    uint32_t real = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int pos = dw * 4 + j, img = pos / PQ, rem = pos - img * PQ, p = rem / Q, q = rem - p * Q;
        h[j] = img < ni ? p * stride - pad : H;   // beyond the last image: outside under every tap
        w[j] = q * stride - pad;
        at[j] = tap_image(img, pitch) + (h[j] * W + w[j]) * E;
        real |= img < ni ? 0x80u << (8 * j) : 0u;
    }
    if (GRAD && c0 == 0 && row0 == 0) *reinterpret_cast<uint32_t *>(mask + m) = real >> 7;
    for (int row = row0; row < cg * taps; row += side) {
        if (GRAD) {
            uint32_t vh = 0, vl = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t v = h[j] < H ? *reinterpret_cast<const uint16_t *>(codes + at[j] + row * HW * 2) : 0u;
                vh |= (v >> 8) << (8 * j);
                vl |= (v & 255u) << (8 * j);
            }
            *reinterpret_cast<uint32_t *>(out + (int64_t)(c0 + row) * len + m) = vh;
            *reinterpret_cast<uint32_t *>(lo + (int64_t)(c0 + row) * len + m) = vl ^ real;
        } else {
            const int c = row / taps, t = row - c * taps, r = t / S, s = t - r * S, off = c * HW + r * W + s;
            uint32_t v = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool in = (unsigned)(h[j] + r) < (unsigned)H && (unsigned)(w[j] + s) < (unsigned)W;
                v |= (in ? (uint32_t)(uint8_t)codes[at[j] + off] : zb) << (8 * j);
            }
            *reinterpret_cast<uint32_t *>(out + ((int64_t)t * channels + c0 + c) * len + m) = v;
        }
    }
}
__global__ __launch_bounds__(kThreads) void tap_operands(const int16_t *__restrict__ g16, const int8_t *__restrict__ x, PadG g, TapG t,
                                                         int S, int taps, const q8t_qparams *__restrict__ qpx, int8_t *__restrict__ A,
                                                         int8_t *__restrict__ X, int8_t *__restrict__ mask)
{
    extern __shared__ __align__(16) int8_t codes[];
    const int n0 = blockIdx.x * t.NI, ni = min(t.NI, g.N - n0), by = blockIdx.y;   // ni < 0 behind the last image
    if (by < t.gblocks) {
        const int c0 = by * t.CGg;
        tap_rows<true>(codes, reinterpret_cast<const int8_t *>(g16), n0, ni, t.NI, g.K, c0, min(t.CGg, g.K - c0), g.P, g.Q, g.P, g.Q, 1, 0, 1,
                       1, t.pitchg, 0, A, g.Mp, A + (int64_t)g.K * g.Mp, mask);
    } else {
        const int c0 = (by - t.gblocks) * t.CGx;
        tap_rows<false>(codes, x, n0, ni, t.NI, g.C, c0, min(t.CGx, g.C - c0), g.H, g.W, g.P, g.Q, g.stride, g.pad, S, taps, t.pitchx,
                        (uint32_t)(qpx->zero_point - (1 << (qpx->bits - 1))) & 255u, X, g.XL, nullptr, nullptr);
    }
}

// ---- C[z][i][j] = sum over slice z of A'[i][m] * B'[j][m] ---------------------------------------
// Also leaves the sums of the staged bytes per row (of A') and per column (row of B') and slice.
// Staging role of a thread (see gemm_core.h): chunk q = tid & 3 of tile rows ar = tid >> 2 and ar + RP.
// the columns of B': channels of the padded input at the offset of a tap
struct Columns {
    int count;                        // columns that exist
    int RS, S, stride, sa, C, PC;
    int64_t pitch;                    // bytes from channel to channel
    __device__ __forceinline__ int64_t offset(int j) const
    {
        j = min(j, count - 1);        // surplus columns of the last tile repeat the last one
        const int c = j / RS, t = j - c * RS, r = t / S, s = t - r * S;
        const int i = r / stride, k = s / stride, cls = (r - i * stride) * sa + (s - k * stride);
        return ((int64_t)cls * C + c) * pitch + i * PC + k;
    }
};

__device__ __forceinline__ uint4 ld16(const int8_t *p)
{
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

struct NtRegs {
    uint4 a0, a1, b0, b1, ones;   // ones: which of the 16 positions are real
};
template <class C>
struct NtOps {
    typedef NtRegs R;
    const int8_t *pa, *pa1, *pb, *pb1, *pm;   // first step: two rows, two columns, the mask
    int64_t at;                               // bytes to the next step
    int stride;                               // from step to step
    bool need_a, need_b;                      // this workgroup reports the row / column sums of its tiles
    int sa0, sa1, sb0, sb1;
    __device__ __forceinline__ void load(R &r, bool valid)
    {
        const int64_t o = valid ? at : 0;
        r.a0 = *reinterpret_cast<const uint4 *>(pa + o);
        r.a1 = *reinterpret_cast<const uint4 *>(pa1 + o);
        r.b0 = ld16(pb + o);
        r.b1 = C::NB == 2 ? ld16(pb1 + o) : r.b0;
        r.ones = *reinterpret_cast<const uint4 *>(pm + o);
        at += stride;
    }
    __device__ __forceinline__ static int masked_sum(const uint4 &v, const uint4 &m, int s)
    {
        s = __builtin_amdgcn_sdot4((int)v.x, (int)m.x, s, false);
        s = __builtin_amdgcn_sdot4((int)v.y, (int)m.y, s, false);
        s = __builtin_amdgcn_sdot4((int)v.z, (int)m.z, s, false);
        return __builtin_amdgcn_sdot4((int)v.w, (int)m.w, s, false);
    }
    __device__ __forceinline__ void prepare(R &r, bool valid)
    {
        // a surplus step stages zero B' rows, so whatever A' holds adds nothing to the products
        r.b0 = q8t_gemm::sel16(valid, r.b0);
        r.b1 = q8t_gemm::sel16(valid, r.b1);
        if (need_a) {   // uniform over the workgroup
            sa0 += valid ? bytesum16(r.a0) : 0;
            sa1 += valid ? bytesum16(r.a1) : 0;
        }
        if (need_b) {
            sb0 = masked_sum(r.b0, r.ones, sb0);
            if (C::NB == 2) sb1 = masked_sum(r.b1, r.ones, sb1);
        }
    }
};

__device__ __forceinline__ int quad_sum(int v)
{
    v += __shfl_xor(v, 1, Q8T_WAVE);
    v += __shfl_xor(v, 2, Q8T_WAVE);
    return v;
}

template <class C>
__device__ __forceinline__ void write_partials(int32_t *__restrict__ dst, int Rbp, int r0, int c0,
                                               const v4i (&acc)[C::MT][C::NT])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, kb = lane >> 4;
    const int rowbase = C::rowbase(wave), colbase = C::colbase(wave);
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < C::NT; ++nt)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                dst[(size_t)(r0 + rowbase + mt * 16 + kb * 4 + j) * Rbp + c0 + colbase + nt * 16 + l16] = acc[mt][nt][j];
}

// The KS groups of C::THREADS threads of a workgroup take every KS-th step of its slice into tiles of their own and add
// them up through LDS: as many wavefronts in flight with 1 / KS of the partial tiles in memory.  96 -> 200 3x3 @27 batch 50,
// 128x128 tiles: 756 workgroups of one group 34.5 us + 9.6 for wgrad_finish (50 MB of partial tiles each way), 252 of two
// 38.5 + 5.7, 512 of two slower by a tenth for every layer with enough steps.  The main loop runs at 0.95 POP/s either way.
template <class C, int KS>
__global__ __launch_bounds__(C::THREADS *KS) void gemm_nt(const int8_t *__restrict__ A, const int8_t *__restrict__ B,
                                                          const int8_t *__restrict__ mask, Columns cols, int rows, int64_t Mp,
                                                          int slice, int Rap, int Rbp, int nz, int32_t *__restrict__ part,
                                                          int *__restrict__ rsum, int *__restrict__ csum)
{
    constexpr int MT = C::MT, NT = C::NT, SHARE = NT / KS;
    extern __shared__ __align__(16) int8_t smem[];

    // logical tile order: row tiles fastest (they share the B' tile), then column tiles (same A' slice)
    const int nx = Rap / C::BM, ny = Rbp / C::BN;
    const int lg = q8t_gemm::xcd_logical(nx * ny * nz);
    if (lg >= nx * ny * nz) return;
    const int bx = lg % nx, by = (lg / nx) % ny, z = lg / (nx * ny);
    const int tid = threadIdx.x % C::THREADS, grp = threadIdx.x / C::THREADS, ar = tid >> 2, q = tid & 3;
    int8_t *sA = smem + grp * C::LDS_BYTES, *sB = sA + 2 * C::BM * 64;
    const int r0 = bx * C::BM, c0 = by * C::BN;
    const int64_t mb = (int64_t)z * slice;
    const int64_t me = mb + slice < Mp ? mb + slice : Mp;
    const int steps = (int)((me - mb) >> 6) / KS;   // Mp and slice are multiples of 64 * KS

    NtOps<C> ops;
    const int64_t first = mb + grp * 64 + q * 16;
    ops.pa = A + (size_t)min(r0 + ar, rows - 1) * Mp + first;   // surplus rows of the last tile repeat the last one
    ops.pa1 = A + (size_t)min(r0 + ar + C::RP, rows - 1) * Mp + first;
    ops.pb = B + cols.offset(c0 + ar) + first;
    ops.pb1 = B + cols.offset(c0 + ar + C::RP) + first;
    ops.pm = mask + first;
    ops.at = 0;
    ops.stride = 64 * KS;
    ops.need_a = by == 0;
    ops.need_b = bx == 0;
    ops.sa0 = ops.sa1 = ops.sb0 = ops.sb1 = 0;

    v4i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (v4i){0, 0, 0, 0};
    q8t_gemm::pipeline<C>(ops, steps, sA, sB, acc, tid);

    // byte sums of this slice: the four threads of a row hold its pieces
    const int sa0 = quad_sum(ops.sa0), sa1 = quad_sum(ops.sa1), sb0 = quad_sum(ops.sb0), sb1 = quad_sum(ops.sb1);
    int *sums = reinterpret_cast<int *>(smem + KS * C::LDS_BYTES);   // [KS][BM + BN]
    if (q == 0) {
        int *s = sums + grp * (C::BM + C::BN);
        s[ar] = sa0;
        s[ar + C::RP] = sa1;
        s[C::BM + ar] = sb0;
        if (C::NB == 2) s[C::BM + ar + C::RP] = sb1;
    }
    // group o adds up column tiles o * SHARE .. of the others
    v4i *fold = reinterpret_cast<v4i *>(smem);   // [owner][KS - 1][MT * SHARE][THREADS]
    __syncthreads();                             // the operand tiles are no longer needed
#pragma unroll
    for (int o = 0; o < KS; ++o)
        if (o != grp) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < SHARE; ++t)
                    fold[((o * (KS - 1) + (grp < o ? grp : grp - 1)) * (MT * SHARE) + mt * SHARE + t) * C::THREADS + tid] =
                        acc[mt][o * SHARE + t];
        }
    __syncthreads();
    if (grp == 0) {
        for (int i = tid; i < C::BM + C::BN; i += C::THREADS) {
            int s = 0;
#pragma unroll
            for (int k = 0; k < KS; ++k) s += sums[k * (C::BM + C::BN) + i];
            if (i < C::BM) {
                if (by == 0) rsum[(size_t)z * Rap + r0 + i] = s;
            } else if (bx == 0) {
                csum[(size_t)z * Rbp + c0 + i - C::BM] = s;
            }
        }
    }
    const int lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kb = lane >> 4;
    int32_t *dst = part + (size_t)z * Rap * Rbp + (size_t)(r0 + C::rowbase(wave) + kb * 4) * Rbp + c0 + C::colbase(wave) + l16;
#pragma unroll
    for (int o = 0; o < KS; ++o)
        if (o == grp) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int t = 0; t < SHARE; ++t) {
                    v4i v = acc[mt][o * SHARE + t];
#pragma unroll
                    for (int k = 0; k < KS - 1; ++k)
                        v += fold[((o * (KS - 1) + k) * (MT * SHARE) + mt * SHARE + t) * C::THREADS + tid];
#pragma unroll
                    for (int j = 0; j < 4; ++j) dst[(size_t)(mt * 16 + j) * Rbp + (o * SHARE + t) * 16] = v[j];
                }
        }
}
template <class C, int KS>
constexpr size_t nt_lds_bytes()
{
    return (size_t)KS * (C::LDS_BYTES + (C::BM + C::BN) * sizeof(int));
}

// ---- 1x1, stride 1, no padding, planes of a multiple of 64 positions ---------------------------
// Both operands are read in place: a step is 64 consecutive positions of one image, where row k
// of the gradient and row c of the input are contiguous in NCHW.  The 16-bit codes are split into
// their byte planes in registers.  A row tile holds RP output channels: its first RP rows are the
// high bytes, the next RP rows the low bytes, and the slice results keep that tiled row order.
template <class C>
struct DirectOps {
    typedef q8t_gemm::Regs R;
    const int16_t *g16;
    const int8_t *x;
    int K, Cin, PQ, cpi, krow, crow, q;
    int n, ch, n_first, ch_first;
    bool need_a, need_b;
    int shi, slo, sb0, sb1;
    __device__ __forceinline__ void load(q8t_gemm::Regs &r, bool valid)
    {
        const int nn = valid ? n : n_first, cc = valid ? ch : ch_first;
        const int16_t *pa = g16 + ((size_t)nn * K + krow) * PQ + cc * 64 + q * 16;
        const int8_t *pb = x + ((size_t)nn * Cin + crow) * PQ + cc * 64 + q * 16;
        r.a0 = *reinterpret_cast<const uint4 *>(pa);
        r.a1 = *reinterpret_cast<const uint4 *>(pa + 8);
        r.b0 = *reinterpret_cast<const uint4 *>(pb);
        r.b1 = C::NB == 2 ? *reinterpret_cast<const uint4 *>(pb + (size_t)C::RP * PQ) : r.b0;
        const bool wrap = ch + 1 == cpi;
        ch = wrap ? 0 : ch + 1;
        n += wrap ? 1 : 0;
    }
    __device__ __forceinline__ void prepare(q8t_gemm::Regs &r, bool valid)
    {
        uint4 hi, lo;
        hi.x = __builtin_amdgcn_perm(r.a0.y, r.a0.x, 0x07050301u);
        hi.y = __builtin_amdgcn_perm(r.a0.w, r.a0.z, 0x07050301u);
        hi.z = __builtin_amdgcn_perm(r.a1.y, r.a1.x, 0x07050301u);
        hi.w = __builtin_amdgcn_perm(r.a1.w, r.a1.z, 0x07050301u);
        lo.x = __builtin_amdgcn_perm(r.a0.y, r.a0.x, 0x06040200u) ^ 0x80808080u;
        lo.y = __builtin_amdgcn_perm(r.a0.w, r.a0.z, 0x06040200u) ^ 0x80808080u;
        lo.z = __builtin_amdgcn_perm(r.a1.y, r.a1.x, 0x06040200u) ^ 0x80808080u;
        lo.w = __builtin_amdgcn_perm(r.a1.w, r.a1.z, 0x06040200u) ^ 0x80808080u;
        r.a0 = hi;
        r.a1 = lo;
        r.b0 = q8t_gemm::sel16(valid, r.b0);   // a surplus step stages zero input rows
        r.b1 = q8t_gemm::sel16(valid, r.b1);
        if (need_a) {   // uniform over the workgroup
            shi += valid ? bytesum16(hi) : 0;
            slo += valid ? bytesum16(lo) : 0;
        }
        if (need_b) {
            sb0 += bytesum16(r.b0);
            if (C::NB == 2) sb1 += bytesum16(r.b1);
        }
    }
};

template <class C>
__global__ __launch_bounds__(C::THREADS, C::MINB) void gemm_direct(const int16_t *__restrict__ g16, const int8_t *__restrict__ x,
                                                                    int K, int Cin, int PQ, int steps_total, int steps_slice,
                                                                    int Rap, int Rbp, int nz, int32_t *__restrict__ part,
                                                                    int *__restrict__ rsum, int *__restrict__ csum)
{
    __shared__ __align__(16) int8_t sA[2 * C::BM * 64];
    __shared__ __align__(16) int8_t sB[2 * C::BN * 64];

    const int nx = K / C::RP, ny = Rbp / C::BN;
    const int lg = q8t_gemm::xcd_logical(blockIdx.x, nx * ny * nz);
    if (lg >= nx * ny * nz) return;
    const int bx = lg % nx, by = (lg / nx) % ny, z = lg / (nx * ny);
    const int tid = threadIdx.x, ar = tid >> 2, q = tid & 3;
    const int r0 = bx * C::BM, c0 = by * C::BN;
    const int t0 = z * steps_slice;
    const int steps = min(steps_slice, steps_total - t0);

    DirectOps<C> ops;
    ops.g16 = g16;
    ops.x = x;
    ops.K = K;
    ops.Cin = Cin;
    ops.PQ = PQ;
    ops.cpi = PQ >> 6;   // steps per image
    ops.q = q;
    ops.krow = bx * C::RP + ar;
    ops.crow = c0 + ar;
    ops.n = ops.n_first = t0 / ops.cpi;
    ops.ch = ops.ch_first = t0 - ops.n * ops.cpi;
    ops.need_a = by == 0;
    ops.need_b = bx == 0;
    ops.shi = ops.slo = ops.sb0 = ops.sb1 = 0;

    v4i acc[C::MT][C::NT];
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < C::NT; ++nt) acc[mt][nt] = (v4i){0, 0, 0, 0};
    q8t_gemm::pipeline<C>(ops, steps, sA, sB, acc, tid);

    const int shi = quad_sum(ops.shi), slo = quad_sum(ops.slo), sb0 = quad_sum(ops.sb0), sb1 = quad_sum(ops.sb1);
    if (by == 0 && q == 0) {
        rsum[(size_t)z * Rap + r0 + ar] = shi;
        rsum[(size_t)z * Rap + r0 + C::RP + ar] = slo;
    }
    if (bx == 0 && q == 0) {
        csum[(size_t)z * Rbp + c0 + ar] = sb0;
        if (C::NB == 2) csum[(size_t)z * Rbp + c0 + ar + C::RP] = sb1;
    }
    write_partials<C>(part + (size_t)z * Rap * Rbp, Rbp, r0, c0, acc);
}

// ---- slices -> exact 64-bit sums -> outputs ------------------------------------------------------
// acc(k,col) = sum (g - zg)(x - zx),  g = 256*hi + lo + 128 :
//   256*S_hi + S_lo + (128 - zg)*colsum - zx*(256*rowsum_hi + rowsum_lo + (128 - zg)*Mp)
// A workgroup owns 256/zgn consecutive outputs; its zgn groups of lanes share the slices.
__global__ __launch_bounds__(kThreads) void wgrad_finish(const int32_t *__restrict__ part, const int *__restrict__ rsum,
                                                         const int *__restrict__ csum, int nz, int K, int CRS, int Rap,
                                                         int Rbp, int64_t Mp, const q8t_qparams *__restrict__ qpg,
                                                         const q8t_qparams *__restrict__ qpx, float *__restrict__ dw,
                                                         int64_t *__restrict__ acc_out, int zgn, int tiled, int S, int GP)
{
    __shared__ long long red[5][kThreads];
    const int per = kThreads / zgn;
    const int o = threadIdx.x % per, zg = threadIdx.x / per;
    const int64_t id = (int64_t)blockIdx.x * per + o;
    const bool ok = id < (int64_t)K * CRS;
    long long shi = 0, slo = 0, rhi = 0, rlo = 0, cs = 0;
    int k = 0, col = 0;
    if (ok) {
        k = (int)(id / CRS);
        col = (int)(id - (int64_t)k * CRS);
        // GP > 0: the partial sums keep the taps of one (channel, filter row) in groups of GP columns
        if (GP) col = (col / S) * GP + col % S;
        // rows of the two byte planes: [all high | all low], or per `tiled` channels [high | low]
        const int rh = tiled ? (k / tiled) * 2 * tiled + (k % tiled) : k, rl = tiled ? rh + tiled : K + k;
        for (int z = zg; z < nz; z += zgn) {
            shi += part[((size_t)z * Rap + rh) * Rbp + col];
            slo += part[((size_t)z * Rap + rl) * Rbp + col];
            rhi += rsum[(size_t)z * Rap + rh];
            rlo += rsum[(size_t)z * Rap + rl];
            cs += csum[(size_t)z * Rbp + col];
        }
    }
    if (zgn > 1) {
        red[0][threadIdx.x] = shi;
        red[1][threadIdx.x] = slo;
        red[2][threadIdx.x] = rhi;
        red[3][threadIdx.x] = rlo;
        red[4][threadIdx.x] = cs;
        __syncthreads();
        if (zg != 0 || !ok) return;
        shi = slo = rhi = rlo = cs = 0;
        for (int g = 0; g < zgn; ++g) {
            shi += red[0][g * per + o];
            slo += red[1][g * per + o];
            rhi += red[2][g * per + o];
            rlo += red[3][g * per + o];
            cs += red[4][g * per + o];
        }
    }
    if (!ok) return;
    const int zsg = qpg->zero_point - (1 << (qpg->bits - 1)), zsx = qpx->zero_point - (1 << (qpx->bits - 1));
    const int64_t ca = 128 - zsg;
    const int64_t v = 256 * shi + slo + ca * cs - (int64_t)zsx * (256 * rhi + rlo + ca * Mp);
    if (acc_out) acc_out[id] = v;
    if (dw) dw[id] = (float)((double)v * (double)(qpg->scale * qpx->scale));
}

struct Plan {
    int P, Q, CRS, Rap, Rbp, nz, slice, direct, taps, ks;
    int cfg;      // 2: 256x256 tiles, 1: 128x128, 0: 128x64
    PadG pad;
    int64_t Mtot, Mp;
    size_t o_B, o_mask, o_part, o_rsum, o_csum, total;
};

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

// ---- weight gradient of a layer with few input channels (the network's first layer), one kernel ----
// GEMM view as above (rows = byte planes of g16 for 64 output channels, columns = (channel, filter
// row) groups of GP taps, reduction = positions), but neither operand is laid out in HBM: a
// workgroup walks output rows (n, p); for each it splits the 64 x Q gradient values into the two
// byte planes straight into the LDS operand tile, stages the R input rows of every channel and
// cuts the column operand out of them (16 consecutive positions of one tap = 16 bytes `stride`
// apart in a staged row), multiplies, and keeps the 128 x Kf accumulator tile in registers until its
// share of the rows is done.  Positions Q..127 of a row hold (0, zero code): they add nothing and
// are counted in the reduction length handed to wgrad_finish.  The loads for the next output row
// are issued before the current one is multiplied.
// Needs: C*R*GP <= 256, stride 1 or 2, Q <= 128 and Q % 16 == 0, W % 4 == 0, 16-byte aligned g16
// rows (Q % 8 == 0), at most UX dwords of input and UA / UB operand pieces per thread and row.
template <int GP, int NT>
__global__ __launch_bounds__(kThreads) void wgrad_smallc(const int16_t *__restrict__ g16, const int8_t *__restrict__ x, int C,
                                                         int H, int W, int R, int S, int stride, int pad, int P, int Q, int K,
                                                         int RB, int rows_total, const q8t_qparams *__restrict__ qpx,
                                                         int32_t *__restrict__ part, int *__restrict__ rsum,
                                                         int *__restrict__ csum)
{
    constexpr int Kf = NT * 16, UX = 6, UA = 4, UB = 5;
    extern __shared__ __align__(16) int8_t lds[];
    int8_t *sA = lds;                                    // [2][128][64]
    int8_t *sB = sA + 2 * 128 * 64;                      // [2][Kf][64]
    int *sums = reinterpret_cast<int *>(sB + 2 * Kf * 64);   // [128] rows of A', [Kf] rows of B'
    int8_t *rows = reinterpret_cast<int8_t *>(sums + 128 + Kf);   // [C*R][Wp] + 16
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kq = lane >> 4;
    const int z = blockIdx.x, kblk = blockIdx.y;
    const int row0 = z * RB, row1 = min(rows_total, row0 + RB);
    const int zx = qpx->zero_point - (1 << (qpx->bits - 1));
    const uint32_t zfill = (uint32_t)(zx & 255) * 0x01010101u;
    const int CR = C * R, L = (pad + 3) & ~3, Wp = (L + W + pad + 3) & ~3;
    const int W4 = W >> 2, Q8 = Q >> 3, Q16 = Q >> 4;

    // ---- fixed roles of the thread ----
    int xd[UX], xr[UX], xo[UX];          // input dwords: LDS offset (-1: none), filter row - pad, offset inside an image
    int ag[UA], ad[UA];                  // gradient pieces of 8 values: offset inside an image, LDS offset (-1: none)
    int bs[UB], bd[UB], bj[UB];          // column pieces of 16 positions: byte offset in `rows`, LDS offset (-1), column
#pragma unroll
    for (int u = 0; u < UX; ++u) {
        const int i = u * kThreads + tid;
        xd[u] = -1;
        xr[u] = xo[u] = 0;
        if (i < CR * W4) {
            const int cr = i / W4, w4 = i - cr * W4, c = cr / R, r = cr - c * R;
            xd[u] = cr * Wp + L + w4 * 4;
            xr[u] = r - pad;
            xo[u] = c * H * W + w4 * 4;
        }
    }
#pragma unroll
    for (int u = 0; u < UA; ++u) {
        const int i = u * kThreads + tid;
        ad[u] = -1;
        ag[u] = 0;
        if (i < 64 * Q8) {
            const int k = i / Q8, ch = i - k * Q8, m = ch * 8;
            ag[u] = (kblk * 64 + k) * P * Q + m;
            ad[u] = (m >> 6) * (128 * 64) + k * 64 + ((((m & 63) >> 4) ^ q8t_gemm::swz(k)) * 16) + ((m >> 3) & 1) * 8;
        }
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
        const int i = u * kThreads + tid;
        bd[u] = -1;
        bs[u] = bj[u] = 0;
        if (i < CR * S * Q16) {
            const int t = i / Q16, c = i - t * Q16, gg = t / S, s2 = t - gg * S, j = gg * GP + s2;
            bj[u] = j;
            bs[u] = gg * Wp + L - pad + s2 + stride * 16 * c;
            bd[u] = (c >> 2) * (Kf * 64) + j * 64 + (((c & 3) ^ q8t_gemm::swz(j)) * 16);
        }
    }
    // ---- LDS: A' zero, B' and the staged rows at the zero code ----
    {
        uint32_t *w = reinterpret_cast<uint32_t *>(sA);
        for (int i = tid; i < (2 * 128 * 64) >> 2; i += kThreads) w[i] = 0;
        w = reinterpret_cast<uint32_t *>(sB);
        for (int i = tid; i < (2 * Kf * 64) >> 2; i += kThreads) w[i] = zfill;
        w = reinterpret_cast<uint32_t *>(rows);
        for (int i = tid; i < (CR * Wp + 16) >> 2; i += kThreads) w[i] = zfill;
        for (int i = tid; i < 128 + Kf; i += kThreads) sums[i] = 0;
    }
    v4i acc[2][NT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (v4i){0, 0, 0, 0};
    int sah[UA], sal[UA], sbs[UB];
#pragma unroll
    for (int u = 0; u < UA; ++u) sah[u] = sal[u] = 0;
#pragma unroll
    for (int u = 0; u < UB; ++u) sbs[u] = 0;

    uint32_t xv[UX];
    uint4 av[UA];
    auto issue = [&](int row) {
        const int n = row / P, p = row - n * P;
        const int8_t *xb = x + (size_t)n * C * H * W;
        const int16_t *gb = g16 + (size_t)n * K * P * Q + (size_t)p * Q;
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            const int h = p * stride + xr[u];
            xv[u] = zfill;
            if (xd[u] >= 0 && (unsigned)h < (unsigned)H) xv[u] = *reinterpret_cast<const uint32_t *>(xb + xo[u] + (size_t)h * W);
        }
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            av[u] = make_uint4(0, 0, 0, 0);
            if (ad[u] >= 0) av[u] = *reinterpret_cast<const uint4 *>(gb + ag[u]);
        }
    };
    if (row0 < row1) issue(row0);
    for (int row = row0; row < row1; ++row) {
        __syncthreads();   // the fill, or the previous row's multiply, is done with sA / sB / rows
#pragma unroll
        for (int u = 0; u < UX; ++u)
            if (xd[u] >= 0) *reinterpret_cast<uint32_t *>(rows + xd[u]) = xv[u];
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            if (ad[u] < 0) continue;
            const uint32_t h0 = __builtin_amdgcn_perm(av[u].y, av[u].x, 0x07050301u);
            const uint32_t h1 = __builtin_amdgcn_perm(av[u].w, av[u].z, 0x07050301u);
            const uint32_t l0 = __builtin_amdgcn_perm(av[u].y, av[u].x, 0x06040200u) ^ 0x80808080u;
            const uint32_t l1 = __builtin_amdgcn_perm(av[u].w, av[u].z, 0x06040200u) ^ 0x80808080u;
            *reinterpret_cast<uint2 *>(sA + ad[u]) = make_uint2(h0, h1);
            *reinterpret_cast<uint2 *>(sA + ad[u] + 64 * 64) = make_uint2(l0, l1);
            sah[u] += bytesum4(h0) + bytesum4(h1);
            sal[u] += bytesum4(l0) + bytesum4(l1);
        }
        if (row + 1 < row1) issue(row + 1);
        __syncthreads();   // staged rows complete
        // column operand: 16 positions of one tap are 16 bytes `stride` apart; read the aligned dwords
        // that contain them, shift to the first byte, keep every stride-th byte
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            if (bd[u] < 0) continue;
            const int a0 = bs[u] & ~3;
            const uint32_t sh = (uint32_t)(bs[u] & 3);
            uint32_t o[4];
            if (stride == 1) {
                uint32_t d[5];
#pragma unroll
                for (int i = 0; i < 5; ++i) d[i] = *reinterpret_cast<const uint32_t *>(rows + a0 + 4 * i);
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = __builtin_amdgcn_alignbyte(d[i + 1], d[i], sh);
            } else {
                uint32_t d[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) d[i] = *reinterpret_cast<const uint32_t *>(rows + a0 + 4 * i);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t e0 = __builtin_amdgcn_alignbyte(d[2 * i + 1], d[2 * i], sh);
                    const uint32_t e1 = __builtin_amdgcn_alignbyte(d[2 * i + 2], d[2 * i + 1], sh);
                    o[i] = __builtin_amdgcn_perm(e1, e0, 0x06040200u);   // bytes 0, 2, 4, 6 of the 8
                }
            }
            *reinterpret_cast<uint4 *>(sB + bd[u]) = make_uint4(o[0], o[1], o[2], o[3]);
            sbs[u] += bytesum4(o[0]) + bytesum4(o[1]) + bytesum4(o[2]) + bytesum4(o[3]);
        }
        __syncthreads();
        // wavefront w multiplies rows [32w, 32w + 32) of A' (w < 2: high plane) against every column tile
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            v4i af[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = wave * 32 + i * 16 + l16;
                af[i] = *reinterpret_cast<const v4i *>(sA + ks * (128 * 64) + r * 64 + ((kq ^ q8t_gemm::swz(r)) * 16));
            }
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int r = nt * 16 + l16;
                const v4i bf = *reinterpret_cast<const v4i *>(sB + ks * (Kf * 64) + r * 64 + ((kq ^ q8t_gemm::swz(r)) * 16));
                acc[0][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[0], bf, acc[0][nt], 0, 0, 0);
                acc[1][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[1], bf, acc[1][nt], 0, 0, 0);
            }
        }
    }
    // ---- byte sums of the rows of A' and B' (zero-point correction), then the partial tile ----
    __syncthreads();
#pragma unroll
    for (int u = 0; u < UA; ++u) {
        if (ad[u] < 0) continue;
        const int k = (u * kThreads + tid) / Q8;
        atomicAdd(&sums[k], sah[u]);
        atomicAdd(&sums[64 + k], sal[u]);
    }
#pragma unroll
    for (int u = 0; u < UB; ++u)
        if (bd[u] >= 0) atomicAdd(&sums[128 + bj[u]], sbs[u]);
    __syncthreads();
    const int Rap = 2 * K;
    if (tid < 128) rsum[(size_t)z * Rap + (tid < 64 ? kblk * 64 + tid : K + kblk * 64 + tid - 64)] = sums[tid];
    // positions Q..127 of every row hold the zero code
    if (kblk == 0 && tid < Kf) csum[(size_t)z * Kf + tid] = sums[128 + tid] + (row1 > row0 ? (row1 - row0) * (128 - Q) * zx : 0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int lr = wave * 32 + i * 16 + kq * 4 + jj;
            const int gr = lr < 64 ? kblk * 64 + lr : K + kblk * 64 + lr - 64;
            int32_t *dst = part + ((size_t)z * Rap + gr) * Kf + l16;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) dst[nt * 16] = acc[i][nt][jj];
        }
}

struct FusedPlan {
    int P, Q, GP, Kf, nz, RB, rows;
    size_t lds, o_rsum, o_csum, total;
};

bool make_fused_plan(const q8t_conv_desc *d, FusedPlan *p)
{
    if (d->N <= 0 || d->C <= 0 || d->C >= 64 || d->K <= 0 || d->K % 64 || d->H <= 0 || d->W <= 0) return false;
    if (d->R <= 0 || d->S <= 0 || d->S > 8 || d->R > 100 || d->stride < 1 || d->stride > 2 || d->pad < 0 || d->pad > 100)
        return false;
    if (d->H + 2 * d->pad < d->R || d->W + 2 * d->pad < d->S || d->W % 4) return false;
    p->P = (d->H + 2 * d->pad - d->R) / d->stride + 1;
    p->Q = (d->W + 2 * d->pad - d->S) / d->stride + 1;
    if (p->Q > 128 || p->Q % 16) return false;
    p->GP = d->S <= 4 ? 4 : 8;
    p->Kf = (d->C * d->R * p->GP + 63) / 64 * 64;
    if (p->Kf > 256) return false;
    const int CR = d->C * d->R, L = (d->pad + 3) & ~3, Wp = (L + d->W + d->pad + 3) & ~3;
    // pieces per thread and output row
    if (CR * (d->W / 4) > kThreads * 6 || 64 * (p->Q / 8) > kThreads * 4 || CR * d->S * (p->Q / 16) > kThreads * 5) return false;
    const int64_t rows = (int64_t)d->N * p->P;
    if (rows >= ((int64_t)1 << 30) || (int64_t)d->N * d->K * p->P * p->Q >= ((int64_t)1 << 31) ||
        (int64_t)d->N * d->C * d->H * d->W >= ((int64_t)1 << 31))
        return false;
    p->rows = (int)rows;
    // two workgroups per compute unit; a workgroup's accumulators take at most 512 rows of 128 products
    int64_t nz = rows < 512 ? rows : 512;
    if ((rows + nz - 1) / nz > 512) nz = (rows + 511) / 512;
    if (nz > 65535) return false;
    p->RB = (int)((rows + nz - 1) / nz);
    p->nz = (int)((rows + p->RB - 1) / p->RB);
    p->lds = (size_t)2 * 128 * 64 + (size_t)2 * p->Kf * 64 + (size_t)(128 + p->Kf) * sizeof(int) + (((size_t)CR * Wp + 15) & ~(size_t)15) + 16;
    if (p->lds > 65536) return false;
    p->o_rsum = up256((size_t)p->nz * 2 * d->K * p->Kf * sizeof(int32_t));
    p->o_csum = p->o_rsum + up256((size_t)p->nz * 2 * d->K * sizeof(int));
    p->total = p->o_csum + up256((size_t)p->nz * p->Kf * sizeof(int));
    return true;
}


// false: more positions than 32 bits count
bool make_padded(const q8t_conv_desc *d, int P, int Q, int64_t step, bool taps, PadG *g)
{
    const int st = d->stride;
    g->N = d->N;
    g->C = d->C;
    g->H = d->H;
    g->W = d->W;
    g->K = d->K;
    g->P = P;
    g->Q = Q;
    g->stride = st;
    g->pad = d->pad;
    // a plane per tap is the case of planes that no two taps share: nothing to pad
    g->ra = taps || d->R < st ? d->R : st;
    g->sa = taps || d->S < st ? d->S : st;
    const int er = taps ? 0 : (d->R - 1) / st, es = taps ? 0 : (d->S - 1) / st;
    // columns (rows) v of a plane are padding on the left where st*v + b < pad, on the right where st*v + b >= W + pad:
    // the last `share` ones of a row are the first ones of the next where both hold for every plane
    auto pitch = [&](int out, int extra, int in, int planes) {
        int share = 0;
        while (share < extra && (int64_t)st * share + planes - 1 < d->pad && (int64_t)st * (out + extra - share - 1) >= in + d->pad) ++share;
        return (int64_t)out + extra - share;
    };
    const int64_t PC = pitch(Q, es, d->W, g->sa), PR = pitch(P, er, d->H, g->ra);
    const int64_t len = (int64_t)d->N * PC * PR;
    if (len + (er + 2) * PC >= ((int64_t)1 << 31) - (1 << 16)) return false;
    g->PC = (int)PC;
    g->IS = (int)(PC * PR);
    g->Mp = (len + step - 1) / step * step;
    g->XL = (g->Mp + er * PC + es + 15) & ~(int64_t)15;   // the last step reads this far under the last tap
    const int64_t chunks = (g->XL + kPadChunk - 1) / kPadChunk, channels = d->K + (int64_t)g->ra * g->sa * d->C;
    // channels per workgroup: the more, the less arithmetic per code, while 2048 workgroups are left; and a launch holds fewer than 2^16
    // blocks of them
    int64_t rows = chunks * channels / 2048;
    rows = rows < 1 ? 1 : (rows > 16 ? 16 : rows);
    if (rows < (channels + 32767) / 32768) rows = (channels + 32767) / 32768;
    g->rows = (int)rows;
    g->gblocks = (int)((d->K + rows - 1) / rows);
    g->xblocks = (int)((d->C + rows - 1) / rows);
    if (g->gblocks + (int64_t)g->ra * g->sa * g->xblocks > 65535) return false;
    g->chunks = (int)chunks;
    return true;
}

// tap_operands: 256 positions a row (a wavefront's store), whole dwords, 60 KB of codes at most; channels while two thousand
// workgroups are left.  false: not the planes it is for, or too large.
bool tap_groups(const PadG &g, TapG *t)
{
    const int64_t PQ = (int64_t)g.P * g.Q, HW = (int64_t)g.H * g.W;
    if (PQ > 3) return false;
    const int unit = PQ == 2 ? 2 : 4;
    constexpr int64_t room = 60 * 1024;
    if (unit * (HW + 8) > room) return false;
    int64_t ni = 256 / PQ / unit * unit;
    while (ni > unit && (ni * (HW + 8) > room || ni >= 2 * (int64_t)g.N)) ni = (ni / 2 + unit - 1) / unit * unit;
    t->NI = (int)ni;
    const int64_t groups = (g.Mp + ni * PQ - 1) / (ni * PQ);
    t->gx = (unsigned)groups;
    size_t lds = 0;
    auto side = [&](int64_t channels, int64_t bytes, int *cgs, int *pitch, int *blocks) {
        int64_t cg = (room / ni - 8) / bytes;
        if (cg > groups * channels / 1024) cg = groups * channels / 1024;
        if (cg < (channels + 32766) / 32767) cg = (channels + 32766) / 32767;
        *cgs = (int)cg;
        *pitch = (int)(((cg * bytes + 3) >> 2 | 1) * 4);
        *blocks = (int)((channels + cg - 1) / cg);
        const size_t need = (size_t)tap_image((int)ni - 1, *pitch) + *pitch;
        if (need > lds) lds = need;
    };
    side(g.K, 2 * PQ, &t->CGg, &t->pitchg, &t->gblocks);
    side(g.C, HW, &t->CGx, &t->pitchx, &t->xblocks);
    t->lds = lds;
    return lds <= 65536 && groups * (t->gblocks + t->xblocks) < (1 << 24);
}

// taps: a plane of the input per tap; ks: groups of wavefronts that share a tile's reduction
bool make_plan(const q8t_conv_desc *d, bool taps, bool groups, Plan *p)
{
    if (d->N <= 0 || d->C <= 0 || d->K <= 0 || d->H <= 0 || d->W <= 0 || d->R <= 0 || d->S <= 0) return false;
    if (d->stride < 1 || d->pad < 0) return false;
    if (d->H + 2 * d->pad < d->R || d->W + 2 * d->pad < d->S) return false;
    p->P = (d->H + 2 * d->pad - d->R) / d->stride + 1;
    p->Q = (d->W + 2 * d->pad - d->S) / d->stride + 1;
    const int64_t crs = (int64_t)d->C * d->R * d->S;
    if (crs > (1 << 24) || d->K > (1 << 22)) return false;
    p->CRS = (int)crs;
    p->Mtot = (int64_t)d->N * p->P * p->Q;
    if (p->Mtot >= ((int64_t)1 << 36)) return false;
    if ((int64_t)d->N * d->C >= ((int64_t)1 << 31) || (int64_t)d->N * d->K >= ((int64_t)1 << 31)) return false;
    p->Rap = (2 * d->K + BM - 1) / BM * BM;
    p->Rbp = (p->CRS + 63) / 64 * 64;
    // 1x1 / stride 1 / no padding on planes of a multiple of 64 positions: operands are used in place
    p->direct = d->R == 1 && d->S == 1 && d->stride == 1 && d->pad == 0 && (p->P * p->Q) % 64 == 0 && d->K % 64 == 0 &&
                d->C % 64 == 0;
    p->cfg = (p->Rap % 256 == 0 && p->Rbp % 256 == 0 && (!p->direct || d->K % 128 == 0)) ? 2 : (p->Rbp % 128 == 0 ? 1 : 0);
    p->taps = taps;
    p->ks = !groups || p->cfg == 2 ? 1 : (p->cfg == 1 ? 2 : 4);
    const int bm = p->cfg == 2 ? 256 : 128, bn = p->cfg == 2 ? 256 : (p->cfg == 1 ? 128 : 64);
    const int64_t tiles = (int64_t)(p->Rap / bm) * (p->Rbp / bn);
    const int64_t step = 64 * p->ks;   // positions that the groups of a workgroup take at a time
    if (!make_padded(d, p->P, p->Q, step, taps, &p->pad)) return false;
    p->Mp = p->pad.Mp;
    // Slices.  The big tile, and the small ones with groups, run one workgroup per compute unit: (just under) a multiple of 256
    // of them; the small tiles without groups, and in place, three.  Laid out: four steps a group or more (two and eight: within 2 us
    // of it over 20 layers, few tiles over few positions better with four, 48 -> 96 3x3 @7 batch 200 24 against 27 us).
    const bool dir = p->direct, three = p->cfg < 2 && (dir || !groups);
    int64_t nz = three ? (768 + tiles - 1) / tiles : (tiles >= 256 ? 1 : 256 / tiles);
    const int64_t least = dir ? 1024 : (three ? 8 : 4) * step, most = (p->Mp + least - 1) / least;   // enough steps per slice
    if (nz > most) nz = most;
    const int64_t ovf = (p->Mp + kMaxSlice - 1) / kMaxSlice;  // 32-bit accumulator bound
    if (nz < ovf) nz = ovf;
    int64_t slice = ((p->Mp + nz - 1) / nz + step - 1) / step * step;
    if (slice > kMaxSlice) slice = kMaxSlice;
    nz = (p->Mp + slice - 1) / slice;
    if (nz > 65535 || tiles * nz >= ((int64_t)1 << 30)) return false;
    p->nz = (int)nz;
    p->slice = (int)slice;
    p->o_B = up256((size_t)2 * d->K * p->Mp);
    p->o_mask = p->o_B + up256((size_t)p->pad.ra * p->pad.sa * d->C * p->pad.XL);
    p->o_part = p->o_mask + up256((size_t)p->Mp);
    p->o_rsum = p->o_part + up256((size_t)p->nz * p->Rap * p->Rbp * sizeof(int32_t));
    p->o_csum = p->o_rsum + up256((size_t)p->nz * p->Rap * sizeof(int));
    p->total = p->o_csum + up256((size_t)p->nz * p->Rbp * sizeof(int));
    return true;
}

// Microseconds of a call by this plan (operands laid out): the operands, the rounds of workgroups and their steps, the partial sums.
// Fitted to 2530 shapes in eight plans each; measured over estimated 0.8 .. 1.2 in 95% of them.
double plan_us(const q8t_conv_desc *d, const Plan &p)
{
    const PadG &g = p.pad;
    const int planes = g.ra * g.sa, PQ = p.P * p.Q;
    const double A = 1e-6 * d->K * g.Mp, X = 1e-6 * planes * d->C * g.XL;
    double us;
    if (p.taps && PQ < 4) {
        us = 8.5 + 1.7 * A + 0.9 * X;
    } else if (PQ < 4) {
        us = 8.0 + 5.0 * A + 2.0 * X;
    } else {
        const double blocks = (double)g.chunks * (d->K + (double)planes * d->C) / g.rows;
        const double x = d->stride > 1 ? 0.55 : (!p.taps || d->R * d->S == 1 ? 0.33 : (p.Q < 4 ? 0.46 : 0.14 + 0.42 / p.Q));
        us = 6.5 + 0.22 * g.rows + 2.3e-3 * blocks + 0.8 * A + x * X;
    }
    const int bm = p.cfg == 2 ? 256 : 128, bn = p.cfg == 2 ? 256 : (p.cfg == 1 ? 128 : 64);
    const int64_t wgs = (int64_t)(p.Rap / bm) * (p.Rbp / bn) * p.nz;
    const int steps = p.slice / (64 * p.ks);
    const bool three = p.cfg < 2 && p.ks == 1;
    const double round = wgs > (three ? 768 : 256) ? wgs / (three ? 768.0 : 256.0) : 1.0;
    if (three) us += round * (p.cfg ? 1.2 + 0.61 * steps : 1.6 + 0.34 * steps);
    else us += round * (p.cfg == 2 ? 5.9 : (p.cfg ? 4.0 : 4.7));
    us += (double)((wgs + 255) / 256) * steps * (three ? (p.cfg ? 0.14 : 0.11) : (p.cfg == 2 ? 0.67 : (p.cfg ? 0.71 : 0.87)));
    return us + 1.5e-6 * p.nz * p.Rap * p.Rbp + 2.4e-6 * d->K * p.CRS;
}

// The plan of a call.  Padded planes hold PC * PR positions where P * Q are real: filters as large as the plane multiply
// mostly zeros (7x7 without padding @7, 512 -> 512 batch 1024 1430 us, with a plane per tap 142); where they hold few, a plane per tap is
// a copy R * S times the input.  Groups of wavefronts that share a tile keep the partial sums small, and leave compute units idle where tiles times slices
// are just above their number (248 -> 512 3x3 @12 batch 18, 280 tiles: 54 us, 45 without).  Over 2530 shapes the plan
// taken is 3.2% slower than the best of the four in the mean, and 1.06 times as fast as padded planes with groups always.  A plane per tap is taken a fifth below the padded planes only
// (its estimate errs more), and up to 2 GB of it.
bool make_plan(const q8t_conv_desc *d, Plan *p)
{
    *p = {};
    const bool first = make_plan(d, false, true, p);
    if (first && p->direct) return true;
    double best = first ? plan_us(d, *p) : 1e30;
    auto consider = [&](bool taps, bool groups, double bias) {
        Plan q;
        if (!make_plan(d, taps, groups, &q) || (taps && best < 1e30 && q.o_mask - q.o_B > ((size_t)1 << 31))) return;
        const double us = plan_us(d, q) * bias;
        if (us < best) {
            best = us;
            *p = q;
        }
    };
    const bool small = first ? p->cfg < 2 : true;
    if (small) consider(false, false, 1 / 0.95);
    if (d->R <= d->stride && d->S <= d->stride && (int64_t)p->P * p->Q >= 4) return best < 1e30;   // the padded planes are planes per tap
    const double bias = (int64_t)p->P * p->Q < 4 ? 1.0 : 1 / 0.8;
    consider(true, true, bias);
    if (small) consider(true, false, bias / 0.95);
    return best < 1e30;
}

}  // namespace

bool q8t_gemm_wgrad_supported(const q8t_conv_desc *d)
{
    Plan p;
    FusedPlan f;
    return make_plan(d, &p) || make_fused_plan(d, &f);
}

size_t q8t_gemm_wgrad_ws(const q8t_conv_desc *d)
{
    Plan p;
    FusedPlan f;
    const size_t a = make_plan(d, &p) ? p.total : 0, b = make_fused_plan(d, &f) ? f.total : 0;
    return a > b ? a : b;
}

int q8t_gemm_wgrad(const q8t_conv_desc *d, const int16_t *g16, const q8t_qparams *qg, const int8_t *x,
                   const q8t_qparams *qx, float *dw, int64_t *acc_out, void *ws, hipStream_t st)
{
    FusedPlan f;
    if (make_fused_plan(d, &f) && q8t_aligned(g16, 16) && q8t_aligned(x, 4)) {
        if (!ws || !q8t_aligned(ws, 16)) return Q8T_ERR_WORKSPACE;
        int32_t *part = (int32_t *)ws;
        int *rsum = (int *)((char *)ws + f.o_rsum);
        int *csum = (int *)((char *)ws + f.o_csum);
        const dim3 grid((unsigned)f.nz, (unsigned)(d->K / 64));
#define Q8T_GO(GPV, NTV)                                                                                              \
    hipLaunchKernelGGL((wgrad_smallc<GPV, NTV>), grid, dim3(kThreads), f.lds, st, g16, x, d->C, d->H, d->W, d->R, d->S, \
                       d->stride, d->pad, f.P, f.Q, d->K, f.RB, f.rows, qx, part, rsum, csum)
        const int nt = f.Kf / 16;
        if (f.GP == 8) {
            if (nt == 4) Q8T_GO(8, 4); else if (nt == 8) Q8T_GO(8, 8); else if (nt == 12) Q8T_GO(8, 12); else Q8T_GO(8, 16);
        } else {
            if (nt == 4) Q8T_GO(4, 4); else if (nt == 8) Q8T_GO(4, 8); else if (nt == 12) Q8T_GO(4, 12); else Q8T_GO(4, 16);
        }
#undef Q8T_GO
        Q8T_LAUNCH_CHECK();
        const int CRS = d->C * d->R * d->S;
        const int64_t count = (int64_t)d->K * CRS;
        const int zgn = f.nz >= 64 ? 16 : (f.nz >= 8 ? 4 : 1);
        const int per = kThreads / zgn;
        hipLaunchKernelGGL(wgrad_finish, dim3((unsigned)((count + per - 1) / per)), dim3(kThreads), 0, st, part, rsum, csum,
                           f.nz, d->K, CRS, 2 * d->K, f.Kf, (int64_t)f.rows * 128, qg, qx, dw, acc_out, zgn, 0, d->S, f.GP);
        Q8T_LAUNCH_CHECK();
        return Q8T_OK;
    }
    Plan p;
    if (!make_plan(d, &p)) return Q8T_ERR_SHAPE;
    if (!ws || !q8t_aligned(ws, 16)) return Q8T_ERR_WORKSPACE;
    int8_t *A = (int8_t *)ws;
    int8_t *B = (int8_t *)ws + p.o_B;
    int32_t *part = (int32_t *)((char *)ws + p.o_part);
    int *rsum = (int *)((char *)ws + p.o_rsum);
    int *csum = (int *)((char *)ws + p.o_csum);
    int8_t *mask = (int8_t *)ws + p.o_mask;
    const Columns cols = {p.CRS, d->R * d->S, d->S, p.taps ? (d->R > d->S ? d->R : d->S) : d->stride, p.pad.sa, d->C, p.pad.PC, p.pad.XL};
    const int direct = p.direct && q8t_aligned(g16, 16) && q8t_aligned(x, 16);
    if (direct) {
        const int steps_total = (int)(p.Mtot >> 6), steps_slice = p.slice >> 6;
#define Q8T_GO(CFG)                                                                                                       \
    hipLaunchKernelGGL(gemm_direct<CFG>, dim3(q8t_gemm::xcd_grid((int64_t)(d->K / CFG::RP) * (p.Rbp / CFG::BN) * p.nz)), \
                       dim3(CFG::THREADS), 0, st, g16, x, d->K, d->C, p.P * p.Q, steps_total, steps_slice, p.Rap, p.Rbp, \
                       p.nz, part, rsum, csum)
        if (p.cfg == 2) Q8T_GO(q8t_gemm::Big);
        else if (p.cfg == 1) Q8T_GO(q8t_gemm::Mid);
        else Q8T_GO(q8t_gemm::Small);
#undef Q8T_GO
        Q8T_LAUNCH_CHECK();
    } else {
        TapG tg;
        if (p.taps && tap_groups(p.pad, &tg)) {
            hipLaunchKernelGGL(tap_operands, dim3(tg.gx, (unsigned)(tg.gblocks + tg.xblocks)), dim3(kThreads), tg.lds, st, g16, x, p.pad, tg,
                               d->S, d->R * d->S, qx, A, B, mask);
        } else {
            const unsigned gy = (unsigned)(p.pad.gblocks + p.pad.ra * p.pad.sa * p.pad.xblocks);
            const unsigned gx = (unsigned)p.pad.chunks < (1u << 23) / gy ? (unsigned)p.pad.chunks : (1u << 23) / gy;
            hipLaunchKernelGGL(pad_operands, dim3(gx, gy), dim3(kThreads), 0, st, g16, x, p.pad, qx, A, B, mask);
        }
        Q8T_LAUNCH_CHECK();
#define Q8T_GO(CFG, KS)                                                                                               \
    {                                                                                                                 \
        static Q8tLdsOptIn optin;                                                                                     \
        constexpr size_t lds = nt_lds_bytes<CFG, KS>();                                                               \
        if (lds > 65536 && q8t_allow_lds(optin, (const void *)gemm_nt<CFG, KS>, lds) != Q8T_OK) return Q8T_ERR_HIP;    \
        hipLaunchKernelGGL((gemm_nt<CFG, KS>), q8t_gemm::xcd_rows((int64_t)(p.Rap / CFG::BM) * (p.Rbp / CFG::BN) * p.nz), \
                           dim3(CFG::THREADS * KS), lds, st, A, B, mask, cols, 2 * d->K, p.Mp, p.slice, p.Rap, p.Rbp, p.nz, \
                           part, rsum, csum);                                                                         \
    }
    if (p.cfg == 2) Q8T_GO(q8t_gemm::Big, 1)
    else if (p.cfg == 1 && p.ks == 2) Q8T_GO(q8t_gemm::Mid, 2)
    else if (p.cfg == 1) Q8T_GO(q8t_gemm::Mid, 1)
    else if (p.ks == 4) Q8T_GO(q8t_gemm::Small, 4)
    else Q8T_GO(q8t_gemm::Small, 1)
#undef Q8T_GO
    Q8T_LAUNCH_CHECK();
    }
    {
        const int64_t count = (int64_t)d->K * p.CRS;
        const int zgn = p.nz >= 64 ? 16 : (p.nz >= 8 ? 4 : 1);   // lanes sharing the slices of one output
        const int per = kThreads / zgn;
        hipLaunchKernelGGL(wgrad_finish, dim3((unsigned)((count + per - 1) / per)), dim3(kThreads), 0, st,
                           part, rsum, csum, p.nz, d->K, p.CRS, p.Rap, p.Rbp, p.Mtot, qg, qx, dw, acc_out, zgn,
                           direct ? (p.cfg == 2 ? 128 : 64) : 0, 1, 0);
        Q8T_LAUNCH_CHECK();
    }
    return Q8T_OK;
}
