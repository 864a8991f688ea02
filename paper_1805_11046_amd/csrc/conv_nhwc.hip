// General MFMA path for the forward and layer-gradient convolutions (Section 4: both products
// take 8-bit operands and accumulate in 32 bits): any filter size, stride, padding and channel count.
// Two launches per call:
//
//  1. prepare      to_nhwc: the NCHW int8 operand is rewritten channel-contiguous ([N][H][W][Cp], Cp = reduction
//                  channels rounded up to 16) into the workspace, so that 16 reduction channels of one
//                  filter tap are one aligned 16-byte piece (to_nhwc_small for many small planes); and
//                  repack_taps: filter -> [class][output channel][tap][Cp], each row filled up with zeros to a multiple
//                  of 64 and the output channels to a multiple of 64, and the per-output-channel sums
//                  (per stride class).
//  2. igemm_nhwc   implicit GEMM, rows = output positions, columns = output channels, K = the pieces of
//                  (tap, 16 channels) eight to a step of 128, which go from memory to LDS without registers
//                  (gemm_core.h; 128x128 or 128x64 tiles).  The sums of the operand rows, which the zero-point
//                  correction needs, are products with ones beside the others.
//
// Until the pieces were copied (registers between memory and LDS, steps of 64, sums per position from a pass of their own, the
// two relayouts one after the other), a whole call took, us, before / now: 128->256 3x3/2 @28 batch 256 forward 68.1 / 63.2, layer
// gradient 84.0 / 72.6; 64->128 3x3/2 @56 batch 32 32.5 / 22.6, 29.2 / 23.2; 96->200 3x3 @27 batch 50 52.4 / 47.2, 50.7 / 40.6;
// 240->240 3x3 @20 batch 200 123 / 106, 112 / 95; 16->16 3x3 @32 batch 128 25.1 / 21.7, 20.0 / 16.2.  Geometric mean over 400
// drawn shapes 1.24 (forward), 1.35 (layer gradient).  Of the 41 us of the first one's product its steps are 20, the rest its
// first loads and its results, which 784 workgroups on 512 places overlap only in part.
//
// Pieces of 16 instead of 64 channels are what lets any channel count run here: 16 channels under a 3x3 filter
// are 9 pieces (3 surplus) where whole steps per tap would be 9 times 4.
// Surplus operand channels are zeros and so are the surplus filter bytes.
//
// Padded taps are staged as the stored zero point, which makes their corrected contribution
// exactly zero; with a = stored code, za/zb = stored zero points:
//    sum (a-za)(b-zb) = sum ab - zb*sum a - za*sum b + Kp*za*zb.
//
// The layer gradient of a strided convolution is split into stride x stride classes of input
// positions (same residue of (h, w) modulo the stride).  Inside a class every position sees the
// same subset of filter taps at stride 1, so each class is a dense problem of its own and no
// multiply is spent on taps that cannot contribute.  All classes run in one launch: the tile index
// selects the class, and the classes of one region, which write interleaved elements of the same
// result lines, are neighbours in the tile order.
#include "q8t_common.h"
#include "q8t_internal.h"
#include "gemm_core.h"

namespace {

using q8t_gemm::v4i;

constexpr int kThreads = 256;
constexpr int MAXT = 49;     // taps (7x7)
constexpr int MAXCLS = 16;   // stride classes (stride <= 4)

struct TapList {             // per tap: two small signed numbers
    int8_t a[MAXT + 3], b[MAXT + 3];
};
struct ClassOffsets {
    int off[MAXCLS + 1];     // taps of class z are [off[z], off[z+1]) of the TapList
};

struct ClassGeo {            // per stride class: positions enumerated, rows, taps and place of its filter rows
    int v[MAXCLS][7];        // OH, OW, M, first tap, number of taps, bytes of a filter row, first filter byte / 64
};
constexpr int CLS_INTS = 8;  // ints per class in the device copy of the table

struct Geo {
    int N, IH, IW, Cp;       // staged operand: [N][IH][IW][Cp], Cp a multiple of 16
    int red;                 // reduction channels (the rest of Cp is padding)
    int OH, OW;              // output positions enumerated by a class (rows m = (n, oh, ow))
    int ish, isw;            // operand step per output step
    int OC, OHf, OWf;        // NCHW result: channels, full height and width
    int OCp;                 // channels rounded up to whole tiles (filter rows, column sums)
    int osh, osw, oph, opw;  // result position = (oh*osh + oph, ow*osw + opw)
    int M;                   // N*OH*OW
    int T;                   // taps of a class
    int vec;                 // result pointers are 16-byte aligned
    int ncls, mtiles;        // stride classes in this launch; row tiles of the largest class
    int fill;                // stride 2, even result size, only class (0, 0) has taps: its workgroups
                             // also write the zeros of the three empty classes
};

// ---- 1. NCHW -> NHWC ---------------------------------------------------------------------------
// A workgroup rewrites 64 positions of one image: tiles of 64 channels x 64 positions go through LDS.  A thread
// takes 4 channels x 4 positions with four 4-byte loads (any alignment), turns them round in registers with eight
// byte permutes and stores 4 dwords, one per position; rows of 21 dwords keep those stores free of bank conflicts
// (20 d mod 64 are sixteen different multiples of 4 for the 16 position quads of a wavefront, its 4 channel quads
// fall between them) and cost the 16-byte reads nothing that shows.  G channel groups of 256 threads share the
// channel tiles of a position where the launch would otherwise be small (few images, small planes).
constexpr int TPITCH = 21;   // dwords
template <int G>
__device__ __forceinline__ void to_nhwc(int block, const int8_t *__restrict__ src, int C, int Cp, int HW, int ptiles,
                                        int8_t *__restrict__ dst)
{
    __shared__ uint32_t tile[G][64 * TPITCH];
    const int n = block / ptiles, p0 = (block - n * ptiles) * 64;
    const int grp = threadIdx.x / kThreads, tid = threadIdx.x % kThreads;
    const int cq = tid >> 4, d = tid & 15;   // staging role: channels 4 cq .., positions 4 d ..
    const int rp = tid >> 2, rq = tid & 3;   // read-out role: position rp, 16-byte chunk rq
    const int ps = p0 + d * 4;
    const int8_t *in = src + (size_t)n * C * HW + ps;
    const int tiles = (Cp + 63) >> 6;
    uint32_t v[4];
    auto load = [&](int c0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = c0 + cq * 4 + i;
            uint32_t w = 0;
            if (c < C) {
                const int8_t *a = in + (size_t)c * HW;
                if (ps + 4 <= HW) {
                    __builtin_memcpy(&w, a, 4);
                } else {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (ps + k < HW) w |= (uint32_t)(uint8_t)a[k] << (8 * k);
                }
            }
            v[i] = w;
        }
    };
    load(grp * 64);
    for (int t = 0; t < tiles; t += G) {   // every group runs the same number of rounds (barriers)
        const int c0 = (t + grp) * 64;
        const uint32_t lo01 = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), hi01 = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
        const uint32_t lo23 = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u), hi23 = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
        uint32_t *w = tile[grp] + d * 4 * TPITCH + cq;
        w[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        w[TPITCH] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        w[2 * TPITCH] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        w[3 * TPITCH] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
        if (t + G < tiles) load(c0 + G * 64);
        __syncthreads();
        const uint32_t *r = tile[grp] + rp * TPITCH + rq * 4;
        const uint4 o = make_uint4(r[0], r[1], r[2], r[3]);
        if (p0 + rp < HW && c0 + rq * 16 < Cp)
            *reinterpret_cast<uint4 *>(dst + ((size_t)n * HW + p0 + rp) * Cp + c0 + rq * 16) = o;
        __syncthreads();
    }
}

// Planes of fewer than 64 positions: the channels of a few neighbouring images are one stretch of the NCHW tensor, and
// their positions one stretch of the copy.  A workgroup takes the images' bytes to LDS as they lie (16-byte loads, any
// alignment) and picks the 16 channels of a position out of it.  With the kernel above a plane costs a workgroup of 64
// positions however small it is: whole 1x1 products over 65536 planes of one position, 48 -> 80 channels 74 -> 23 us,
// 256 -> 512 190 -> 63, of four positions, 64 -> 64 95 -> 40; 4096 planes of 49, 64 -> 64 49 both.
constexpr int kSmallBytes = 32 * 1024;
__device__ __forceinline__ void to_nhwc_small(int block, const int8_t *__restrict__ src, int N, int C, int Cp, int HW, int ipw,
                                              int8_t *__restrict__ dst)
{
    extern __shared__ __align__(16) int8_t flat[];   // [images][C][HW]
    const int n0 = block * ipw, images = min(ipw, N - n0), CC = Cp >> 4;
    const int bytes = images * C * HW, positions = images * HW;
    const int8_t *in = src + (size_t)n0 * C * HW;
    for (int i = threadIdx.x * 16; i < bytes; i += kThreads * 16) {
        if (i + 16 <= bytes) {
            uint4 v;
            __builtin_memcpy(&v, in + i, 16);
            *reinterpret_cast<uint4 *>(flat + i) = v;
        } else {
            for (int k = i; k < bytes; ++k) flat[k] = in[k];
        }
    }
    __syncthreads();
    int8_t *out = dst + (size_t)n0 * HW * Cp;
    for (int i = threadIdx.x; i < positions * CC; i += kThreads) {
        const int pos = i / CC, q = i - pos * CC, img = pos / HW, p = pos - img * HW;
        const int8_t *b = flat + (img * C + q * 16) * HW + p;
        const int left = C - q * 16;   // channels from here on
        uint32_t w[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            w[d] = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * d + e < left) w[d] |= (uint32_t)(uint8_t)b[(4 * d + e) * HW] << (8 * e);
        }
        *reinterpret_cast<uint4 *>(out + (size_t)i * 16) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// ---- filter -> [class][output channel][tap][reduction channel], sums per output channel ------
// One row (output channel j, class z) by THREADS threads; tid: the thread among them, part [THREADS / 64] and stap [MAXT]: their LDS.
// which 0: out = k, reduction = c;  which 1: out = c, reduction = k.
// The first one also writes the tables of the main kernel: operand offsets of the taps (dh in the low half), the classes, and
// three pieces of 16 bytes for what lies outside: the zero code, the zero code in the last piece of a tap (only the channels that
// are there, as the row sums count them), zeros.
constexpr int PADS = MAXT + 3;   // ints from the tap table to those pieces

__device__ __forceinline__ void pad_pieces(int tid, int8_t *pads, int red, const q8t_qparams *__restrict__ qpa)
{
    const int i = tid, last = red & 15, za = qpa->zero_point - (1 << (qpa->bits - 1));
    if (i < 48) pads[i] = i < 16 || (i < 32 && (last == 0 || i - 16 < last)) ? (int8_t)za : (int8_t)0;
}

template <int THREADS>
__device__ __forceinline__ void repack_taps(int tid, int *part, int *stap, int j, int z, int ncls, const int8_t *__restrict__ w,
                                            int Kf, int Cf, int R, int S, int which, int Cp, const TapList &taps, const TapList &offs, const ClassOffsets &co,
                                            const ClassGeo &cg, const q8t_qparams *__restrict__ qpa, int OCp,
                                            int8_t *__restrict__ wt, int *__restrict__ colsum, int *__restrict__ tapoff,
                                            int *__restrict__ clsinfo)
{
    const int OC = which == 0 ? Kf : Cf, red = which == 0 ? Cf : Kf;
    if (j == 0 && z == 0) {
        for (int t = tid; t < co.off[MAXCLS]; t += THREADS)
            tapoff[t] = (int)((uint32_t)(uint16_t)(int16_t)offs.a[t] | ((uint32_t)(uint16_t)(int16_t)offs.b[t] << 16));
        for (int c = tid; c < ncls; c += THREADS)
            for (int k = 0; k < 7; ++k) clsinfo[c * CLS_INTS + k] = cg.v[c][k];
        pad_pieces(tid, reinterpret_cast<int8_t *>(tapoff + PADS), red, qpa);
    }
    const int RS = R * S, t0 = co.off[z], T = co.off[z + 1] - t0, pitch = cg.v[z][5];
    int8_t *out = wt + (size_t)cg.v[z][6] * 64 + (size_t)j * pitch;
    // one loop over (tap, channel): tap by tap, 49 taps of 16 channels were 49 dependent rounds with 16 threads at work
    for (int t = tid; t < T; t += THREADS) stap[t] = taps.a[t0 + t] * S + taps.b[t0 + t];
    __syncthreads();
    int sum = 0;
    for (int i = tid; i < T * Cp; i += THREADS) {
        const int t = i / Cp, c = i - t * Cp;
        int8_t v = 0;
        if (j < OC && c < red) {
            const size_t f = which == 0 ? (size_t)j * Cf + c : (size_t)c * Cf + j;
            v = w[f * RS + stap[t]];
        }
        out[i] = v;
        sum += v;
    }
    if (tid < pitch - T * Cp) out[T * Cp + tid] = 0;   // fewer than 64 bytes
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, Q8T_WAVE);
    if ((tid & 63) == 0) part[tid >> 6] = sum;
    __syncthreads();
    if (tid == 0) {
        int s = 0;
#pragma unroll
        for (int i = 0; i < THREADS / 64; ++i) s += part[i];
        colsum[z * OCp + j] = s;
    }
}

// Both in one launch, the filter rows first: neither needs the other, and the filter alone is 4.8 us.
// G: channel groups of to_nhwc, 0 for to_nhwc_small.  A workgroup of four groups takes one filter row with all of its threads or,
// `apart`, one with each group.  Thousands of short rows (strided layer gradients have a row per class) wait for workgroups to come
// and go, few long ones for the loads of a group: apart up to a mean of 2 bytes a row for every row there is.  Whole calls, one row /
// four rows a workgroup, us: layer gradients 512 <- 128 3x3/4 @2x53 batch 8 (8192 rows of 72 bytes) 33.3 / 16.4, 320 <- 128 5x3/4 @13
// batch 12 (5120 of 120) 30 / 20; 128 <- 256 5x5 @24 batch 5 (128 of 6400) 40.5 / 50.4.  1114 calls: 0.2% slower than the better one.
struct PrepArgs {
    const int8_t *x, *w;
    int8_t *xn, *wt;
    const q8t_qparams *qpa;
    int *colsum, *tapoff, *clsinfo;
    int N, C, Cp, HW, per, ncls, OCp, Kf, Cf, R, S, which;   // per: 64-position tiles of a plane / images a workgroup
    int row0, rows;                                          // first filter row, workgroups of filter rows in this launch
    int apart;                                               // G > 1: G rows a workgroup
    TapList taps, offs;
    ClassOffsets co;
    ClassGeo cg;
};
template <int G>
__global__ __launch_bounds__(kThreads * (G ? G : 1)) void prepare(const PrepArgs p)
{
    constexpr int GROUPS = G ? G : 1;
    __shared__ int part[GROUPS * (kThreads / 64)], stap[GROUPS * MAXT];
    const int b = (int)blockIdx.x - p.rows;
    if (b < 0 && GROUPS > 1 && p.apart) {
        const int grp = threadIdx.x / kThreads, row = p.row0 + (int)blockIdx.x * GROUPS + grp, z = row / p.OCp, j = row - z * p.OCp;
        repack_taps<kThreads>(threadIdx.x % kThreads, part + grp * (kThreads / 64), stap + grp * MAXT, j, z, p.ncls, p.w, p.Kf, p.Cf, p.R,
                              p.S, p.which, p.Cp, p.taps, p.offs, p.co, p.cg, p.qpa, p.OCp, p.wt, p.colsum, p.tapoff, p.clsinfo);
    } else if (b < 0) {
        const int row = p.row0 + (int)blockIdx.x, z = row / p.OCp, j = row - z * p.OCp;
        repack_taps<kThreads * GROUPS>(threadIdx.x, part, stap, j, z, p.ncls, p.w, p.Kf, p.Cf, p.R, p.S, p.which, p.Cp, p.taps, p.offs,
                                       p.co, p.cg, p.qpa, p.OCp, p.wt, p.colsum, p.tapoff, p.clsinfo);
    } else if constexpr (G == 0)
        to_nhwc_small(b, p.x, p.N, p.C, p.Cp, p.HW, p.per, p.xn);
    else
        to_nhwc<G>(b, p.x, p.C, p.Cp, p.HW, p.per, p.xn);
}

// ---- 2. implicit GEMM ---------------------------------------------------------------------------
// The pieces of a step of 128 as a thread of the Dma tiles copies them: piece (tid & 7) ^ perm of the rows tid >> 3 and 64 further
// down, of both operands.  Eight pieces on per step.
template <class C>
struct DmaConvOps {
    const int8_t *xin, *wt, *pads;       // wt: the thread's piece of its filter row
    const __attribute__((address_space(3))) int *stap;
    int IH, IW, Cp, CC, dt, dc;
    size_t wrows;                        // bytes from a filter row to the one 64 further down
    int an[2], ih[2], iw[2];             // image (-1: no such row) and top-left operand position of the two rows
    int lt, lc;                          // tap and piece of it in the next step
    int at, taps, pitch;                 // its place in the reduction, the bytes of the class's taps and of a filter row
    int wave;

    __device__ __forceinline__ void start(const Geo &g, int m0, int n0, int M, int OHW, int OW, int T, int pitch_, const int8_t *wbase, int tid)
    {
        const int r = tid >> 3, q = (tid & 7) ^ C::perm(r);
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        IH = g.IH;
        IW = g.IW;
        Cp = g.Cp;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int m = m0 + r + u * 64, n = m / OHW, rem = m - n * OHW, oh = rem / OW;
            an[u] = m < M ? n : -1;
            ih[u] = oh * g.ish;
            iw[u] = (rem - oh * OW) * g.isw;
        }
        CC = Cp >> 4;
        dt = 8 / CC;
        dc = 8 - dt * CC;
        filter(wbase + (size_t)(n0 + r) * pitch_, T, pitch_, q);
    }
    // from the first piece of a filter on
    __device__ __forceinline__ void filter(const int8_t *row, int T, int pitch_, int q)
    {
        wt = row + q * 16;
        wrows = (size_t)64 * pitch_;
        at = q * 16;
        taps = T * Cp;
        pitch = pitch_;
        lt = q / CC;
        lc = q - lt * CC;
    }
    __device__ __forceinline__ void issue(int8_t *buf)
    {
        const bool in = at < taps;
        const int to = stap[in ? lt : 0];
        const int dh = (int)(int16_t)(to & 0xFFFF), dw = to >> 16;
        const int8_t *out = pads + (!in ? 32 : (lc == CC - 1 ? 16 : 0));
        int8_t *dst = buf + wave * 1024;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int h = ih[u] + dh, w = iw[u] + dw;
            const bool ok = in && an[u] >= 0 && (unsigned)h < (unsigned)IH && (unsigned)w < (unsigned)IW;
            const int8_t *p = xin + (size_t)((an[u] * IH + h) * IW + w) * Cp + lc * 16;
            q8t_gemm::copy16_to_lds(ok ? p : out, dst + u * 8192);
        }
#pragma unroll
        for (int u = 0; u < C::NB; ++u)
            q8t_gemm::copy16_to_lds(at < pitch ? wt + u * wrows : pads + 32, dst + C::BM * C::DK + u * 8192);
        wt += C::DK;
        at += C::DK;
        lc += dc;
        const bool wrap = lc >= CC;
        lc -= wrap ? CC : 0;
        lt += dt + (wrap ? 1 : 0);
    }
};

template <class C>
constexpr size_t conv_lds_bytes()
{
    return (size_t)C::LDS_BYTES + C::BM * (sizeof(long long) + sizeof(int)) + (MAXT + 3) * sizeof(int);
}

template <class C>
__global__ __launch_bounds__(C::THREADS, C::MINB) void igemm_nhwc(const int8_t *__restrict__ xin,
                                                                   const int8_t *__restrict__ wt,
                                                                   const int *__restrict__ colsum,
                                                                   const q8t_qparams *__restrict__ qpa,
                                                                   const q8t_qparams *__restrict__ qpb, Geo g,
                                                                   const int *__restrict__ tapoff,
                                                                   const int *__restrict__ clsinfo,
                                                                   float *__restrict__ out_f, int32_t *__restrict__ out_acc,
                                                                   Q8tConvStat *__restrict__ bnpart)
{
    constexpr int MT = C::MT, NT = C::NT, BM = C::BM, BN = C::BN;
    extern __shared__ __align__(16) int8_t smem[];
    long long *roff = reinterpret_cast<long long *>(smem + C::LDS_BYTES);
    int *rs = reinterpret_cast<int *>(roff + BM);
    int *stap = rs + BM;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kb = lane >> 4;
    // logical tile order: output-channel tiles fastest (they share the operand rows), then the stride
    // classes of one row tile: they write interleaved elements of the same result lines, and run
    // back to back on one XCD so that its L2 merges them before they go to memory
    const int ny = g.OCp / BN, total = g.mtiles * g.ncls * ny;
    const int lg = q8t_gemm::xcd_logical(total);
    if (lg >= total) return;
    const int n0 = (lg % ny) * BN, zc = (lg / ny) % g.ncls, m0 = (lg / (ny * g.ncls)) * BM;
    int wpitch;
    const int8_t *pads;
    {
        const int *ci = clsinfo + zc * CLS_INTS;
        g.OH = ci[0];
        g.OW = ci[1];
        g.M = ci[2];
        g.T = ci[4];
        g.oph = zc / g.osw;
        g.opw = zc - g.oph * g.osw;
        wpitch = ci[5];
        wt += (size_t)ci[6] * 64;
        pads = reinterpret_cast<const int8_t *>(tapoff + PADS);
        tapoff += ci[3];
        colsum += (size_t)zc * g.OCp;
    }
    if (m0 >= g.M) return;   // a smaller class: the whole workgroup leaves before any barrier
    const int za = qpa->zero_point - (1 << (qpa->bits - 1)), zb = qpb->zero_point - (1 << (qpb->bits - 1));
    const float sc = qpa->scale * qpb->scale;
    const int OHW = g.OH * g.OW;

    if (tid < MAXT + 3) stap[tid] = tid < g.T ? tapoff[tid] : 0;
    __syncthreads();
    DmaConvOps<C> ops;
    ops.stap = (const __attribute__((address_space(3))) int *)stap;
    ops.xin = xin;
    ops.pads = pads;
    ops.start(g, m0, n0, g.M, OHW, g.OW, g.T, wpitch, wt, tid);
    if (wpitch) ops.issue(smem);
    // offset of the row's position inside one output channel plane
    if (tid < BM) {
        const int m = m0 + tid;
        long long off = -1;
        if (m < g.M) {
            const int n = m / OHW, rem = m - n * OHW;
            const int oh = rem / g.OW, ow = rem - oh * g.OW;
            off = (long long)n * g.OC * g.OHf * g.OWf + (long long)(oh * g.osh + g.oph) * g.OWf + ow * g.osw + g.opw;
        }
        roff[tid] = off;
    }

    const int colbase = C::colbase(wave);
    v4i acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (v4i){0, 0, 0, 0};

    v4i rsum;
    q8t_gemm::dma_pipeline<C, false>(ops, wpitch >> 6, smem, acc, rsum, tid);
    if (l16 == 0) *reinterpret_cast<v4i *>(&rs[C::row(wave, 0) + kb * 4]) = rsum;
    __syncthreads();

    // ---- epilogue: zero-point correction in wrapping 32-bit arithmetic (the corrected value fits
    // by contract), dequantization; a lane holds 4 consecutive rows of one output channel ----
    const uint32_t kzz = (uint32_t)(g.T * g.red) * (uint32_t)za * (uint32_t)zb;
    const long long plane = (long long)g.OHf * g.OWf;
    uint32_t csn[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) csn[nt] = (uint32_t)za * (uint32_t)colsum[n0 + colbase + nt * 16 + l16];
    // statistics of the lane's output channels over its rows, for the Range BN behind a forward product
    long long st_s[NT];
    int st_mn[NT], st_mx[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        st_s[nt] = 0;
        st_mn[nt] = 2147483647;
        st_mx[nt] = -2147483647 - 1;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int r0 = C::row(wave, mt) + kb * 4;
        long long o[4];
        uint32_t t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = roff[r0 + j];
            t[j] = kzz - (uint32_t)zb * (uint32_t)rs[r0 + j];
        }
        if (g.fill) {
            // result positions (2*oh, 2*ow): the lane's four rows are 8 consecutive floats of result row
            // 2*oh when they share an image row, and row 2*oh + 1 is all zeros
            const bool run = g.vec && o[0] >= 0 && o[1] == o[0] + 2 && o[2] == o[0] + 4 && o[3] == o[0] + 6;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if (n0 + colbase + nt * 16 + l16 >= g.OC) continue;
                const long long cb = (long long)(n0 + colbase + nt * 16 + l16) * plane;
                int c[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) c[j] = (int)((uint32_t)acc[mt][nt][j] + t[j] - csn[nt]);
                if (run && (((o[0] + cb) & 3) == 0)) {
                    const long long b0 = o[0] + cb, b1 = b0 + g.OWf;   // OWf is even: b1 is 8-byte aligned
                    if (out_acc) {
                        *reinterpret_cast<int4 *>(out_acc + b0) = make_int4(c[0], 0, c[1], 0);
                        *reinterpret_cast<int4 *>(out_acc + b0 + 4) = make_int4(c[2], 0, c[3], 0);
                        *reinterpret_cast<int2 *>(out_acc + b1) = make_int2(0, 0);
                        *reinterpret_cast<int2 *>(out_acc + b1 + 2) = make_int2(0, 0);
                        *reinterpret_cast<int2 *>(out_acc + b1 + 4) = make_int2(0, 0);
                        *reinterpret_cast<int2 *>(out_acc + b1 + 6) = make_int2(0, 0);
                    }
                    if (out_f) {
                        *reinterpret_cast<float4 *>(out_f + b0) = make_float4(sc * (float)c[0], 0.f, sc * (float)c[1], 0.f);
                        *reinterpret_cast<float4 *>(out_f + b0 + 4) = make_float4(sc * (float)c[2], 0.f, sc * (float)c[3], 0.f);
                        *reinterpret_cast<float2 *>(out_f + b1) = make_float2(0.f, 0.f);
                        *reinterpret_cast<float2 *>(out_f + b1 + 2) = make_float2(0.f, 0.f);
                        *reinterpret_cast<float2 *>(out_f + b1 + 4) = make_float2(0.f, 0.f);
                        *reinterpret_cast<float2 *>(out_f + b1 + 6) = make_float2(0.f, 0.f);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (o[j] < 0) continue;
                        const long long b = o[j] + cb;
                        if (out_acc) {
                            out_acc[b] = c[j];
                            out_acc[b + 1] = 0;
                            out_acc[b + g.OWf] = 0;
                            out_acc[b + g.OWf + 1] = 0;
                        }
                        if (out_f) {
                            out_f[b] = sc * (float)c[j];
                            out_f[b + 1] = 0.f;
                            out_f[b + g.OWf] = 0.f;
                            out_f[b + g.OWf + 1] = 0.f;
                        }
                    }
                }
            }
            continue;
        }
        const bool contig = g.vec && o[0] >= 0 && o[1] == o[0] + 1 && o[2] == o[0] + 2 && o[3] == o[0] + 3;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (n0 + colbase + nt * 16 + l16 >= g.OC) continue;
            const long long cb = (long long)(n0 + colbase + nt * 16 + l16) * plane;
            int c[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) c[j] = (int)((uint32_t)acc[mt][nt][j] + t[j] - csn[nt]);
            if (bnpart) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (o[j] >= 0) {
                        st_s[nt] += c[j];
                        st_mn[nt] = min(st_mn[nt], c[j]);
                        st_mx[nt] = max(st_mx[nt], c[j]);
                    }
            }
            if (contig && (((o[0] + cb) & 3) == 0)) {
                if (out_acc) *reinterpret_cast<int4 *>(out_acc + o[0] + cb) = make_int4(c[0], c[1], c[2], c[3]);
                if (out_f) {
                    float4 f;
                    f.x = sc * (float)c[0];
                    f.y = sc * (float)c[1];
                    f.z = sc * (float)c[2];
                    f.w = sc * (float)c[3];
                    *reinterpret_cast<float4 *>(out_f + o[0] + cb) = f;
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (o[j] < 0) continue;
                    if (out_acc) out_acc[o[j] + cb] = c[j];
                    if (out_f) out_f[o[j] + cb] = sc * (float)c[j];
                }
            }
        }
    }
    if (bnpart) {
        // fold the lanes that share a channel through LDS slots (the operand tiles are no longer needed)
        unsigned long long *slot_s = reinterpret_cast<unsigned long long *>(smem);
        int *slot_mn = reinterpret_cast<int *>(slot_s + BN), *slot_mx = slot_mn + BN;
        __syncthreads();
        if (tid < BN) {
            slot_s[tid] = 0;
            slot_mn[tid] = 2147483647;
            slot_mx[tid] = -2147483647 - 1;
        }
        __syncthreads();
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int ch = colbase + nt * 16 + l16;
            atomicAdd(&slot_s[ch], (unsigned long long)st_s[nt]);
            atomicMin(&slot_mn[ch], st_mn[nt]);
            atomicMax(&slot_mx[ch], st_mx[nt]);
        }
        __syncthreads();
        if (tid < BN) {
            const int k = n0 + tid;
            Q8tConvStat r;
            r.sum = (long long)slot_s[tid];
            r.mn = slot_mn[tid];
            r.mx = slot_mx[tid];
            bnpart[((size_t)(k >> 6) * g.mtiles + m0 / BM) * 64 + (k & 63)] = r;
        }
    }
}

// ---- layer gradient at stride 2: the two stride classes (ph, 0) and (ph, 1) in one workgroup -----
// Both classes enumerate the same positions (n, oh, ow) when the result width is even, and their
// results are neighbours in memory: (2*oh + ph, 2*ow) and (2*oh + ph, 2*ow + 1).  A workgroup runs the
// main loop once per class into two accumulator sets and writes 8-byte pairs (32-byte runs where a
// lane's four rows share an image row) instead of isolated 4-byte elements, which is what the L2
// request rate of a stride class on its own is bound by.
template <class C>
constexpr size_t conv_pair_lds_bytes()
{
    return conv_lds_bytes<C>() + C::BM * sizeof(int);
}

template <class C>
__global__ __launch_bounds__(C::THREADS, C::MINB) void igemm_nhwc_pair(const int8_t *__restrict__ xin,
                                                                  const int8_t *__restrict__ wt,
                                                                  const int *__restrict__ colsum,
                                                                  const q8t_qparams *__restrict__ qpa,
                                                                  const q8t_qparams *__restrict__ qpb, Geo g,
                                                                  const int *__restrict__ tapoff,
                                                                  const int *__restrict__ clsinfo,
                                                                  float *__restrict__ out_f, int32_t *__restrict__ out_acc)
{
    constexpr int MT = C::MT, NT = C::NT, BM = C::BM, BN = C::BN;
    extern __shared__ __align__(16) int8_t smem[];
    long long *roff = reinterpret_cast<long long *>(smem + C::LDS_BYTES);
    int *rsA = reinterpret_cast<int *>(roff + BM);
    int *rsB = rsA + BM;
    int *stap = rsB + BM;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kb = lane >> 4;
    // logical tile order: output-channel tiles fastest, then the two row parities of one row tile
    const int ny = g.OCp / BN, total = g.mtiles * 2 * ny;
    const int lg = q8t_gemm::xcd_logical(total);
    if (lg >= total) return;
    const int n0 = (lg % ny) * BN, ph = (lg / ny) & 1, m0 = (lg / (ny * 2)) * BM;
    const int *ciA = clsinfo + (ph * 2) * CLS_INTS, *ciB = ciA + CLS_INTS;
    const int OH = ciA[0], OW = ciA[1], M = ciA[2];
    const int TA = ciA[4], TB = ciB[4];
    if (m0 >= M) return;   // the whole workgroup leaves before any barrier
    const int za = qpa->zero_point - (1 << (qpa->bits - 1)), zb = qpb->zero_point - (1 << (qpb->bits - 1));
    const float sc = qpa->scale * qpb->scale;
    const int OHW = OH * OW;

    // the taps of the two classes are neighbours in the table
    if (tid < MAXT + 3) stap[tid] = tid < TA + TB ? tapoff[ciA[3] + tid] : 0;
    __syncthreads();
    DmaConvOps<C> ops;
    ops.stap = (const __attribute__((address_space(3))) int *)stap;
    ops.xin = xin;
    ops.pads = reinterpret_cast<const int8_t *>(tapoff + PADS);
    ops.start(g, m0, n0, M, OHW, OW, TA, ciA[5], wt + (size_t)ciA[6] * 64, tid);
    if (ciA[5]) ops.issue(smem);
    if (tid < BM) {
        const int m = m0 + tid;
        long long off = -1;
        if (m < M) {
            const int n = m / OHW, rem = m - n * OHW;
            const int oh = rem / OW, ow = rem - oh * OW;
            off = (long long)n * g.OC * g.OHf * g.OWf + (long long)(oh * 2 + ph) * g.OWf + ow * 2;
        }
        roff[tid] = off;
    }

    const int colbase = C::colbase(wave);
    v4i accA[MT][NT], accB[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) accA[mt][nt] = accB[mt][nt] = (v4i){0, 0, 0, 0};

    v4i rsumA, rsumB;
    q8t_gemm::dma_pipeline<C, true>(ops, ciA[5] >> 6, smem, accA, rsumA, tid);
    {
        const int r = tid >> 3;
        ops.filter(wt + (size_t)ciB[6] * 64 + (size_t)(n0 + r) * ciB[5], TB, ciB[5], (tid & 7) ^ C::perm(r));
        ops.stap += TA;
    }
    q8t_lds_barrier();   // every wavefront is past its reads of the first class's tiles
    if (ciB[5]) ops.issue(smem);
    q8t_gemm::dma_pipeline<C, true>(ops, ciB[5] >> 6, smem, accB, rsumB, tid);
    if (l16 == 0) {
        *reinterpret_cast<v4i *>(&rsA[C::row(wave, 0) + kb * 4]) = rsumA;
        *reinterpret_cast<v4i *>(&rsB[C::row(wave, 0) + kb * 4]) = rsumB;
    }
    __syncthreads();

    // ---- epilogue: both classes corrected and dequantized, written as pairs ----
    const uint32_t kzzA = (uint32_t)(TA * g.red) * (uint32_t)za * (uint32_t)zb;
    const uint32_t kzzB = (uint32_t)(TB * g.red) * (uint32_t)za * (uint32_t)zb;
    const long long plane = (long long)g.OHf * g.OWf;
    const int *colA = colsum + (size_t)(ph * 2) * g.OCp, *colB = colA + g.OCp;
    uint32_t csA[NT], csB[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        csA[nt] = (uint32_t)za * (uint32_t)colA[n0 + colbase + nt * 16 + l16];
        csB[nt] = (uint32_t)za * (uint32_t)colB[n0 + colbase + nt * 16 + l16];
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int r0 = C::row(wave, mt) + kb * 4;
        long long o[4];
        uint32_t tA[4], tB[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = roff[r0 + j];
            tA[j] = kzzA - (uint32_t)zb * (uint32_t)rsA[r0 + j];
            tB[j] = kzzB - (uint32_t)zb * (uint32_t)rsB[r0 + j];
        }
        const bool run = g.vec && o[0] >= 0 && o[1] == o[0] + 2 && o[2] == o[0] + 4 && o[3] == o[0] + 6;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (n0 + colbase + nt * 16 + l16 >= g.OC) continue;
            const long long cb = (long long)(n0 + colbase + nt * 16 + l16) * plane;
            int a[4], b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[j] = (int)((uint32_t)accA[mt][nt][j] + tA[j] - csA[nt]);
                b[j] = (int)((uint32_t)accB[mt][nt][j] + tB[j] - csB[nt]);
            }
            if (run && (((o[0] + cb) & 3) == 0)) {
                if (out_acc) {
                    *reinterpret_cast<int4 *>(out_acc + o[0] + cb) = make_int4(a[0], b[0], a[1], b[1]);
                    *reinterpret_cast<int4 *>(out_acc + o[0] + cb + 4) = make_int4(a[2], b[2], a[3], b[3]);
                }
                if (out_f) {
                    *reinterpret_cast<float4 *>(out_f + o[0] + cb) =
                        make_float4(sc * (float)a[0], sc * (float)b[0], sc * (float)a[1], sc * (float)b[1]);
                    *reinterpret_cast<float4 *>(out_f + o[0] + cb + 4) =
                        make_float4(sc * (float)a[2], sc * (float)b[2], sc * (float)a[3], sc * (float)b[3]);
                }
            } else if (g.vec) {   // even result width and plane: every pair is 8-byte aligned
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (o[j] < 0) continue;
                    if (out_acc) *reinterpret_cast<int2 *>(out_acc + o[j] + cb) = make_int2(a[j], b[j]);
                    if (out_f) *reinterpret_cast<float2 *>(out_f + o[j] + cb) = make_float2(sc * (float)a[j], sc * (float)b[j]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (o[j] < 0) continue;
                    if (out_acc) {
                        out_acc[o[j] + cb] = a[j];
                        out_acc[o[j] + cb + 1] = b[j];
                    }
                    if (out_f) {
                        out_f[o[j] + cb] = sc * (float)a[j];
                        out_f[o[j] + cb + 1] = sc * (float)b[j];
                    }
                }
            }
        }
    }
}

// Stage the R input rows under output row p of image n, for every channel, into LDS:
// rows[(c*R + r)*pitch + L + w] = x[n][c][p*stride + r - pad][w], the zero code everywhere else
// (padding rows and columns).  L = pad rounded up to a multiple of 4 and pitch a multiple of 4, so
// that aligned dwords of the input are aligned dwords of a staged row.  All loads of a pass are
// issued before the first LDS store: a workgroup's input is a few KB and the pass would otherwise
// be a chain of exposed memory latencies.
__device__ __forceinline__ void stage_rows(const int8_t *__restrict__ x, int n, int C, int H, int W, int R, int stride,
                                           int pad, int p, int L, int pitch, int za, bool vec4, int8_t *rows)
{
    constexpr int U = 6;
    const int CR = C * R, tid = threadIdx.x;
    {
        uint32_t *r32 = reinterpret_cast<uint32_t *>(rows);
        const uint32_t fill = (uint32_t)(za & 255) * 0x01010101u;
        for (int i = tid; i < (CR * pitch) >> 2; i += kThreads) r32[i] = fill;
    }
    __syncthreads();
    if (vec4) {
        const int W4 = W >> 2, items = CR * W4;
        for (int i0 = 0; i0 < items; i0 += kThreads * U) {
            uint32_t v[U];
            int dst[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * kThreads + tid;
                dst[u] = -1;
                v[u] = 0;
                if (i < items) {
                    const int cr = i / W4, w4 = i - cr * W4, c = cr / R, r = cr - c * R;
                    const int h = p * stride + r - pad;
                    if ((unsigned)h < (unsigned)H) {
                        v[u] = *reinterpret_cast<const uint32_t *>(x + (((size_t)n * C + c) * H + h) * W + w4 * 4);
                        dst[u] = cr * pitch + L + w4 * 4;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (dst[u] >= 0) *reinterpret_cast<uint32_t *>(rows + dst[u]) = v[u];
        }
    } else {
        const int items = CR * W;
        for (int i0 = 0; i0 < items; i0 += kThreads * U) {
            int8_t v[U];
            int dst[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * kThreads + tid;
                dst[u] = -1;
                v[u] = 0;
                if (i < items) {
                    const int cr = i / W, w = i - cr * W, c = cr / R, r = cr - c * R;
                    const int h = p * stride + r - pad;
                    if ((unsigned)h < (unsigned)H) {
                        v[u] = x[(((size_t)n * C + c) * H + h) * W + w];
                        dst[u] = cr * pitch + L + w;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (dst[u] >= 0) rows[dst[u]] = v[u];
        }
    }
}

// ---- forward with few input channels and many taps ------------------------------------------------
// The reduction (c, r, s) of an output position is laid out explicitly: xn[m][Kc] with Kc = C*R*S rounded up to a multiple of
// 64, entry c*R*S + r*S + s = the input code under that tap (zero code in the padding and in the surplus columns), plus
// the row sum.  With the filter as [K][Kc] (zeros in the surplus columns) the product is a 1x1 problem for igemm_nhwc.  Beyond
// the limits of the path above (filters of more than 49 taps, strides beyond 4), and where the estimate is lowest here:
// 8 channels under 5x5 taps are 4 K-steps of 64 instead of 7 (8 -> 64 @12 batch 16 20.3 -> 14.2 us, 20 -> 512 7x7/2 34.2 -> 25.6).
// One workgroup per (image, output row): the R input rows of every channel go to LDS once.
__global__ __launch_bounds__(kThreads) void im2col_positions(const int8_t *__restrict__ x, int C, int H, int W, int R, int S,
                                                             int stride, int pad, int P, int Q, int Kc,
                                                             const q8t_qparams *__restrict__ qpx,
                                                             int8_t *__restrict__ xn, int vec4)
{
    extern __shared__ __align__(16) int8_t lds[];
    const int CRS = C * R * S;
    const int L = (pad + 3) & ~3, Wp = (L + W + pad + 3) & ~3;   // staged row: left margin, pitch
    int8_t *rows = lds;                                   // [C*R][Wp]
    int *lut = reinterpret_cast<int *>(lds + ((C * R * Wp + 15) & ~15));   // [Kc]: offset of column j in `rows`, -1: surplus
    const int n = blockIdx.y, p = blockIdx.x, tid = threadIdx.x;
    const int zsx = qpx->zero_point - (1 << (qpx->bits - 1));
    stage_rows(x, n, C, H, W, R, stride, pad, p, L, Wp, zsx, vec4 != 0, rows);
    for (int j = tid; j < Kc; j += kThreads) {
        int off = -1;
        if (j < CRS) {
            const int c = j / (R * S), t = j - c * R * S, r = t / S, s2 = t - r * S;
            off = (c * R + r) * Wp + L - pad + s2;
        }
        lut[j] = off;
    }
    __syncthreads();
    const int chunks = Kc >> 4;
    const size_t m0 = ((size_t)n * P + p) * Q;
    const uint32_t zb = (uint32_t)(zsx & 255);
    for (int it = tid; it < Q * chunks; it += kThreads) {
        const int q = it / chunks, ch = it - q * chunks;
        const int base = q * stride;
        uint32_t w4[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t v = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int off = lut[ch * 16 + d * 4 + e];
                const uint32_t b = off >= 0 ? (uint32_t)(uint8_t)rows[off + base] : zb;
                v |= b << (8 * e);
            }
            w4[d] = v;
        }
        *reinterpret_cast<uint4 *>(xn + (m0 + q) * Kc + ch * 16) = make_uint4(w4[0], w4[1], w4[2], w4[3]);
    }
}

// filter [K][C*R*S] -> [K][Kc] with zero surplus columns, sums per output channel, tap offset 0
__global__ __launch_bounds__(kThreads) void repack_flat(const int8_t *__restrict__ w, int CRS, int Kc, int OH, int OW,
                                                        int M, const q8t_qparams *__restrict__ qpx, int8_t *__restrict__ wt,
                                                        int *__restrict__ colsum, int *__restrict__ tapoff,
                                                        int *__restrict__ clsinfo)
{
    __shared__ int part[kThreads / 64];
    const int k = blockIdx.x;
    if (k == 0) pad_pieces(threadIdx.x, reinterpret_cast<int8_t *>(tapoff + PADS), Kc, qpx);
    int sum = 0;
    for (int j = threadIdx.x; j < Kc; j += kThreads) {
        const int8_t v = j < CRS ? w[(size_t)k * CRS + j] : (int8_t)0;
        wt[(size_t)k * Kc + j] = v;
        sum += v;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, Q8T_WAVE);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        colsum[k] = part[0] + part[1] + part[2] + part[3];
        if (k == 0) {
            tapoff[0] = 0;
            clsinfo[0] = OH;
            clsinfo[1] = OW;
            clsinfo[2] = M;
            clsinfo[3] = 0;
            clsinfo[4] = 1;
            clsinfo[5] = Kc;
            clsinfo[6] = 0;
        }
    }
}

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

struct Plan {
    int red, oc;          // reduction and output channels
    int Cp, OCp;          // rounded up to pieces of 16 / tiles of 64
    int IH, IW;           // operand spatial size
    int OHf, OWf;         // result spatial size
    int ncls;             // stride classes
    size_t o_wt, o_colsum, o_tapoff, o_cls, total;
};

// Operand planes for to_nhwc_small: from half the images on that fill the chip with workgroups of to_nhwc.  Fewer leave
// the latter the shorter chain (512 channels of 49 positions, 64 images: 19.4 against 24.4 us a call), and so do planes of
// many bytes (512 channels of 25 positions, 4096 images: 86 against 91).
bool small_planes(const Plan &p, int N)
{
    const int64_t HW = (int64_t)p.IH * p.IW;
    return HW < 64 && HW * p.red <= 6144 && N >= 1024;
}

bool make_plan(int which, const q8t_conv_desc *d, Plan *p)
{
    if (which < 0 || which > 1) return false;
    if (d->N <= 0 || d->C <= 0 || d->K <= 0 || d->H <= 0 || d->W <= 0 || d->R <= 0 || d->S <= 0) return false;
    if (d->stride < 1 || d->stride > 4 || d->pad < 0 || d->pad > 100) return false;
    if (d->R * d->S > MAXT || d->R > 100 || d->S > 100) return false;
    if (d->H + 2 * d->pad < d->R || d->W + 2 * d->pad < d->S) return false;
    const int P = (d->H + 2 * d->pad - d->R) / d->stride + 1, Q = (d->W + 2 * d->pad - d->S) / d->stride + 1;
    p->red = which == 0 ? d->C : d->K;
    p->oc = which == 0 ? d->K : d->C;
    p->Cp = (p->red + 15) & ~15;
    p->OCp = (p->oc + 63) & ~63;
    p->IH = which == 0 ? d->H : P;
    p->IW = which == 0 ? d->W : Q;
    p->OHf = which == 0 ? P : d->H;
    p->OWf = which == 0 ? Q : d->W;
    p->ncls = which == 0 ? 1 : d->stride * d->stride;
    const int64_t ipos = (int64_t)d->N * p->IH * p->IW, opos = (int64_t)d->N * p->OHf * p->OWf;
    if (ipos >= ((int64_t)1 << 31) || opos >= ((int64_t)1 << 31)) return false;
    if ((int64_t)d->N * (which == 0 ? d->C : d->K) >= ((int64_t)1 << 31)) return false;
    // a launch holds fewer than 2^32 threads: 256 for 64 positions of a plane (to_nhwc)
    if (!small_planes(*p, d->N) && (int64_t)d->N * (((int64_t)p->IH * p->IW + 63) / 64) >= (1 << 24)) return false;
    if (opos >= ((int64_t)1 << 30)) return false;
    p->o_wt = up256((size_t)ipos * p->Cp);
    // filter rows: the taps of a class times Cp, filled up to 64
    const int64_t wbytes = (int64_t)p->OCp * ((int64_t)d->R * d->S * p->Cp + 63 * p->ncls);
    if (wbytes >= ((int64_t)1 << 36) || (int64_t)d->R * d->S * p->Cp >= ((int64_t)1 << 30)) return false;
    p->o_colsum = p->o_wt + up256((size_t)wbytes);
    p->o_tapoff = p->o_colsum + up256((size_t)p->ncls * p->OCp * sizeof(int));
    p->o_cls = p->o_tapoff + up256(PADS * sizeof(int) + 48);
    p->total = p->o_cls + up256((size_t)MAXCLS * CLS_INTS * sizeof(int));
    return true;
}

// Tile: 128x128 from a tile for every compute unit on, else 128x64.  Whole calls with 128x64 / 128x128 tiles, us: 128->256 3x3/2
// @28 batch 256 (784 tiles) 72 / 68, layer gradient 82 / 74; 96->200 3x3 @27 batch 50 (570) 52.4 / 51.5; 256->512 3x3/2 @14
// batch 256 (392) 71 / 61; 48->96 3x3 @24 batch 64 (288) 25.9 / 25.7; 64->128 3x3/2 @56 batch 32 (196) 28.0 / 27.8; 128->256
// 3x3/2 @28 batch 32 (98) 25.0 / 27.5; 256->512 3x3/2 @14 batch 32 (52) 30.8 / 34.4, layer gradient 36 / 41.
bool wide_tiles(int64_t M, int ncls, int OCp)
{
    return OCp % 128 == 0 && (M + 127) / 128 * ncls * (OCp / 128) >= 256;
}

struct SmallPlan {
    int P, Q, Kc;
    size_t lds, o_wt, o_colsum, o_tapoff, total;
};

// forward only: fewer than 64 input channels, output channels a multiple of 64
bool make_small_plan(int which, const q8t_conv_desc *d, SmallPlan *p)
{
    if (which != 0) return false;
    if (d->N <= 0 || d->C <= 0 || d->C >= 64 || d->K <= 0 || d->K % 64 || d->H <= 0 || d->W <= 0) return false;
    if (d->R <= 0 || d->S <= 0 || d->R > 100 || d->S > 100 || d->stride < 1 || d->pad < 0 || d->pad > 100) return false;
    if (d->H + 2 * d->pad < d->R || d->W + 2 * d->pad < d->S) return false;
    const int64_t crs = (int64_t)d->C * d->R * d->S;
    if (crs > 1024) return false;
    p->Kc = (int)((crs + 63) / 64 * 64);
    p->P = (d->H + 2 * d->pad - d->R) / d->stride + 1;
    p->Q = (d->W + 2 * d->pad - d->S) / d->stride + 1;
    if (d->N > 65535 || p->P >= (1 << 24) || d->K >= (1 << 24)) return false;   // 2^32 threads are too many for a launch
    const int64_t M = (int64_t)d->N * p->P * p->Q;
    if (M >= ((int64_t)1 << 31) || (int64_t)d->N * d->C * d->H >= ((int64_t)1 << 31)) return false;
    p->lds = (((size_t)d->C * d->R * ((((d->pad + 3) & ~3) + d->W + d->pad + 3) & ~3) + 15) & ~(size_t)15) +
             (size_t)p->Kc * sizeof(int);
    if (p->lds > 65536) return false;
    p->o_wt = up256((size_t)M * p->Kc);
    p->o_colsum = p->o_wt + up256((size_t)d->K * p->Kc);
    p->o_tapoff = p->o_colsum + up256((size_t)d->K * sizeof(int));
    p->total = p->o_tapoff + 256;
    return true;
}

}  // namespace

bool q8t_smallc_conv_supported(int which, const q8t_conv_desc *d)
{
    SmallPlan p;
    return make_small_plan(which, d, &p);
}

// As q8t_generic_conv_us, for the forward product here (the shape is supported): three launches; 1024 workgroups of the im2col
// side by side, its rows written and read, the K-steps as in q8t_nhwc_conv_us.  Measured time 0.84 .. 1.3 of it in
// 96% of the 200 calls that it was fitted to.
double q8t_smallc_conv_us(const q8t_conv_desc *d, bool stats)
{
    SmallPlan p;
    if (!make_small_plan(0, d, &p)) return 0.0;
    const double M = (double)d->N * p.P * p.Q, wgs = (double)d->N * p.P, rounds = wgs > 1024 ? wgs / 1024 : 1.0;
    const int bn = wide_tiles((int64_t)M, 1, d->K) ? 128 : 64, pitch = ((d->pad + 3) & ~3) + d->W + d->pad;
    const double tiles = (double)(((int64_t)M + 127) / 128) * (d->K / bn);
    const double t = (double)(((int64_t)tiles + 255) / 256) * (bn == 128 ? 1.6 : 1.0);
    const int pieces = (p.Q * (p.Kc / 16) + kThreads - 1) / kThreads;
    const int loads = (d->C * d->R * (d->W % 4 ? d->W : d->W / 4) + kThreads * 6 - 1) / (kThreads * 6);
    const int fill = (d->C * d->R * pitch / 4 + kThreads - 1) / kThreads, steps = p.Kc / 64;
    const double us = 7.6 + 0.33 * steps + 0.28 * steps * (t - 1.0) + 2.6 * t + rounds * (0.1 * pieces + 1.05 * loads + 0.8 * fill) +
                      1.1e-6 * M * p.Kc + 4.4e-6 * d->K * p.Kc;
    return us + (stats ? q8t_range_bn_stats_us(d->N, d->K, (int64_t)p.P * p.Q) : 0.0);
}

size_t q8t_smallc_conv_ws(int which, const q8t_conv_desc *d)
{
    SmallPlan p;
    return make_small_plan(which, d, &p) ? p.total : 0;
}

int q8t_smallc_conv(const q8t_conv_desc *d, const void *a, const q8t_qparams *qa, const void *b, const q8t_qparams *qb,
                    float *out_f, void *out_acc, void *ws, hipStream_t st)
{
    SmallPlan p;
    if (!make_small_plan(0, d, &p)) return Q8T_ERR_SHAPE;
    if (!ws || !q8t_aligned(ws, 16)) return Q8T_ERR_WORKSPACE;
    int8_t *xn = (int8_t *)ws;
    int8_t *wt = (int8_t *)ws + p.o_wt;
    int *colsum = (int *)((char *)ws + p.o_colsum);
    int *tapoff = (int *)((char *)ws + p.o_tapoff);
    const int vec4 = d->W % 4 == 0 && q8t_aligned(a, 4);
    int *clsinfo = tapoff + 8;   // the tap table of this path has one entry
    hipLaunchKernelGGL(repack_flat, dim3((unsigned)d->K), dim3(kThreads), 0, st, (const int8_t *)b, d->C * d->R * d->S, p.Kc,
                       p.P, p.Q, d->N * p.P * p.Q, qa, wt, colsum, tapoff, clsinfo);
    Q8T_LAUNCH_CHECK();
    hipLaunchKernelGGL(im2col_positions, dim3((unsigned)p.P, (unsigned)d->N), dim3(kThreads), p.lds, st, (const int8_t *)a,
                       d->C, d->H, d->W, d->R, d->S, d->stride, d->pad, p.P, p.Q, p.Kc, qa, xn, vec4);
    Q8T_LAUNCH_CHECK();
    Geo g;
    g.N = d->N;
    g.IH = p.P;
    g.IW = p.Q;
    g.Cp = g.red = p.Kc;   // surplus columns hold the zero code
    g.OH = p.P;
    g.OW = p.Q;
    g.ish = g.isw = 1;
    g.OC = g.OCp = d->K;
    g.OHf = p.P;
    g.OWf = p.Q;
    g.osh = g.osw = 1;
    g.oph = g.opw = 0;
    g.M = d->N * p.P * p.Q;
    g.T = 1;
    g.vec = q8t_aligned(out_f, 16) && q8t_aligned(out_acc, 16);
    g.ncls = 1;
    g.fill = 0;
#define Q8T_GO(CFG)                                                                                                   \
    {                                                                                                                 \
        static Q8tLdsOptIn optin;                                                                                     \
        if (conv_lds_bytes<CFG>() > 65536 &&                                                                          \
            q8t_allow_lds(optin, (const void *)igemm_nhwc<CFG>, conv_lds_bytes<CFG>()) != Q8T_OK)                      \
            return Q8T_ERR_HIP;                                                                                       \
        g.mtiles = (g.M + CFG::BM - 1) / CFG::BM;                                                                     \
        const int64_t tiles = (int64_t)g.mtiles * (d->K / CFG::BN);                                                   \
        hipLaunchKernelGGL(igemm_nhwc<CFG>, q8t_gemm::xcd_rows(tiles), dim3(CFG::THREADS), conv_lds_bytes<CFG>(), \
                           st, xn, wt, colsum, qa, qb, g, tapoff, clsinfo, out_f, (int32_t *)out_acc,         \
                           (Q8tConvStat *)nullptr);                                                                \
    }
    if (wide_tiles(g.M, 1, d->K)) Q8T_GO(q8t_gemm::Dma<128>)
    else Q8T_GO(q8t_gemm::Dma<64>)
#undef Q8T_GO
    Q8T_LAUNCH_CHECK();
    return Q8T_OK;
}

bool q8t_nhwc_conv_supported(int which, const q8t_conv_desc *d)
{
    Plan p;
    return make_plan(which, d, &p);
}

size_t q8t_nhwc_conv_ws(int which, const q8t_conv_desc *d)
{
    Plan p;
    return make_plan(which, d, &p) ? p.total : 0;
}

// As q8t_generic_conv_us, for the product here (the shape is supported): two launches, the copy, the filter, then the longest
// class's K-steps (two classes one after the other where a workgroup has both), the first round of them at the price of its latency.
// Isolated results (strides beyond 2; stride 2 on rows of odd length, which have no pairs) cost their lines several times, the more the
// shorter the rows are (256 <- 7 1x1/2 @5 batch 3510 7 us a million, @160 2.5); under 1x1 filters those of narrow or odd rows cost a
// workgroup's end more.  Fitted to half of 20000 layer gradients with a stride, 0.75 .. 1.3 in 90% of the others.
double q8t_nhwc_conv_us(int which, const q8t_conv_desc *d, bool stats)
{
    Plan p;
    if (!make_plan(which, d, &p)) return 0.0;
    const int st = which == 0 ? 1 : d->stride, taps = d->R * d->S, Q = (d->W + st - 1) / st;
    const bool fill = st == 2 && taps == 1 && d->pad == 0 && d->H % 2 == 0 && d->W % 2 == 0;
    const bool pair = st == 2 && !fill && d->W % 2 == 0;
    const int launched = fill ? 1 : (pair ? 2 : p.ncls);
    const int64_t opos = (int64_t)d->N * p.OHf * p.OWf, M = (opos + p.ncls - 1) / p.ncls;
    const int bn = wide_tiles(M, launched, p.OCp) ? 128 : 64;
    const double t = (double)(((M + 127) / 128 * launched * (p.OCp / bn) + 255) / 256) * (bn == 128 ? 1.6 : 1.0), results = 1e-6 * opos * p.oc;
    const int steps = (((d->R + st - 1) / st) * (pair ? d->S : (d->S + st - 1) / st) * p.Cp + 63) / 64;
    const double scatter = st > 2 ? 4.1 : (d->W % 2 ? 2.4 : 0.7) + (taps > 3 ? 0.6 : 0.0), line = st > 2 ? 7.6 : (d->W % 2 ? 11.4 : 7.1);
    double us = 8.2 + 0.28 * steps + 0.16 * steps * (t - 1.0) + 0.75 * t + 0.65e-6 * d->N * p.IH * p.IW * p.Cp +
                4.7e-6 * taps * p.OCp * p.Cp + (st == 1 ? 1.1 : scatter + line / (d->W + 2)) * results;
    if (st > 1 && taps == 1 && Q > 1 && results >= 0.05 && (Q % 4 || (!fill && (d->W % 2 || st > 2)))) us += d->C < 192 ? d->C / 38.0 : 5.0;
    return us + (stats ? 2.9 + 0.54 * results : 0.0);
}

size_t q8t_nhwc_conv_stats_ws(const q8t_conv_desc *d)
{
    Plan p;
    if (!make_plan(0, d, &p)) return 0;
    // one partial per (128-row tile, output channel); larger tiles need fewer
    const int64_t M = (int64_t)d->N * p.OHf * p.OWf;
    return (size_t)((M + 127) / 128) * p.OCp * sizeof(Q8tConvStat);
}

int q8t_nhwc_conv(int which, const q8t_conv_desc *d, const void *a, const q8t_qparams *qa, const void *b,
                  const q8t_qparams *qb, float *out_f, void *out_acc, float *bn_stats, void *stats_ws, void *ws,
                  hipStream_t st)
{
    Plan p;
    if (!make_plan(which, d, &p)) return Q8T_ERR_SHAPE;
    if (!ws || !q8t_aligned(ws, 16)) return Q8T_ERR_WORKSPACE;
    if (bn_stats && (which != 0 || !stats_ws || !q8t_aligned(stats_ws, 16))) return Q8T_ERR_WORKSPACE;
    Q8tConvStat *bnp = bn_stats ? (Q8tConvStat *)stats_ws : (Q8tConvStat *)nullptr;
    int8_t *xn = (int8_t *)ws;
    int8_t *wt = (int8_t *)ws + p.o_wt;
    int *colsum = (int *)((char *)ws + p.o_colsum);
    int *tapoff = (int *)((char *)ws + p.o_tapoff);

    // 1. taps of every class.  forward: one class with all taps, operand offset (r - pad, s - pad).
    // layer gradient: class (ph, pw) keeps the taps with (ph + pad - r) and (pw + pad - s) divisible
    // by the stride; the operand (output-gradient) offset is that quotient.
    TapList rs_list = {}, off_list = {};
    ClassOffsets co = {};
    const int stv = d->stride;
    int nt = 0;
    for (int z = 0; z < p.ncls; ++z) {
        co.off[z] = nt;
        const int ph = z / stv, pw = z % stv;
        for (int r = 0; r < d->R; ++r)
            for (int s = 0; s < d->S; ++s) {
                int dh, dw;
                if (which == 0) {
                    dh = r - d->pad;
                    dw = s - d->pad;
                } else {
                    const int eh = ph + d->pad - r, ew = pw + d->pad - s;
                    if (eh % stv || ew % stv) continue;
                    dh = eh / stv;
                    dw = ew / stv;
                }
                rs_list.a[nt] = (int8_t)r;
                rs_list.b[nt] = (int8_t)s;
                off_list.a[nt] = (int8_t)dh;
                off_list.b[nt] = (int8_t)dw;
                ++nt;
            }
    }
    for (int z = p.ncls; z <= MAXCLS; ++z) co.off[z] = nt;
    // positions of every class
    ClassGeo cg = {};
    int maxM = 0;
    int64_t wrow0 = 0;   // first byte of the class's filter rows / 64
    for (int z = 0; z < p.ncls; ++z) {
        int oh = p.OHf, ow = p.OWf;
        if (which == 1) {
            const int ph = z / stv, pw = z % stv;
            oh = (p.OHf - ph + stv - 1) / stv;
            ow = (p.OWf - pw + stv - 1) / stv;
        }
        const int m = oh > 0 && ow > 0 ? d->N * oh * ow : 0;
        cg.v[z][0] = oh;
        cg.v[z][1] = ow;
        cg.v[z][2] = m;
        cg.v[z][3] = co.off[z];
        cg.v[z][4] = co.off[z + 1] - co.off[z];
        cg.v[z][5] = (cg.v[z][4] * p.Cp + 63) & ~63;
        cg.v[z][6] = (int)wrow0;
        wrow0 += (int64_t)p.OCp * cg.v[z][5] / 64;
        if (m > maxM) maxM = m;
    }
    // stride 2 with taps in class (0, 0) only (a 1x1 filter without padding) and an even result size:
    // that class's workgroups write the zeros of the other three as well
    bool fill = which == 1 && stv == 2 && p.OHf % 2 == 0 && p.OWf % 2 == 0 && cg.v[0][4] > 0;
    for (int z = 1; z < p.ncls; ++z) fill = fill && cg.v[z][4] == 0;
    const int ncls = fill ? 1 : p.ncls;
    if (fill) maxM = cg.v[0][2];
    int *clsinfo = (int *)((char *)ws + p.o_cls);

    // 2. operand and filter relayout
    const int HW = p.IH * p.IW, ptiles = (HW + 63) / 64;
    PrepArgs pa = {};
    pa.x = (const int8_t *)a;
    pa.w = (const int8_t *)b;
    pa.xn = xn;
    pa.wt = wt;
    pa.qpa = qa;
    pa.colsum = colsum;
    pa.tapoff = tapoff;
    pa.clsinfo = clsinfo;
    pa.N = d->N;
    pa.C = p.red;
    pa.Cp = p.Cp;
    pa.HW = HW;
    pa.per = ptiles;
    pa.ncls = p.ncls;
    pa.OCp = p.OCp;
    pa.Kf = d->K;
    pa.Cf = d->C;
    pa.R = d->R;
    pa.S = d->S;
    pa.which = which;
    pa.taps = rs_list;
    pa.offs = off_list;
    pa.co = co;
    pa.cg = cg;
    int64_t blocks = (int64_t)ptiles * d->N;   // of the operand; below 2^31: so is the number of positions
    const bool small = small_planes(p, d->N);
    size_t lds = 0;
    if (small) {
        // images per workgroup: a piece of 16 bytes for every thread, more of them while the launch stays large
        const int plane = p.red * HW, pieces = HW * (p.Cp >> 4);
        int64_t ipw = (kThreads + pieces - 1) / pieces;
        while (d->N / ipw > 2048) ipw *= 2;
        if (ipw > kSmallBytes / plane) ipw = kSmallBytes / plane;   // LDS
        if (ipw > 2048 / HW) ipw = 2048 / HW;
        lds = (size_t)(ipw * plane + 15) & ~(size_t)15;
        pa.per = (int)ipw;
        blocks = (d->N + ipw - 1) / ipw;
    }
    // a launch holds fewer than 2^32 threads: very many filter rows go ahead in launches of their own
    const int64_t rows = (int64_t)p.OCp * p.ncls, room = 1 << 21;
    pa.rows = (int)(rows < room ? rows : room);
    for (; pa.row0 + room < rows; pa.row0 += (int)room) {
        hipLaunchKernelGGL(prepare<0>, dim3((unsigned)room), dim3(kThreads), 0, st, pa);
        Q8T_LAUNCH_CHECK();
    }
    pa.rows = (int)(rows - pa.row0);
    if (blocks + pa.rows >= (1 << 24)) {
        hipLaunchKernelGGL(prepare<0>, dim3((unsigned)pa.rows), dim3(kThreads), 0, st, pa);
        Q8T_LAUNCH_CHECK();
        pa.rows = 0;
    }
    // four channel groups per position tile where single ones would leave wavefront slots empty (256 compute
    // units hold 2048 workgroups of 256 threads)
    const bool four = !small && p.Cp > 64 && blocks < 1024;
    pa.apart = four && (int64_t)d->R * d->S * p.Cp <= 2 * rows * p.ncls;   // bytes of a row, in the mean
    if (pa.apart) pa.rows /= 4;   // a multiple of 64
    const dim3 grid((unsigned)(blocks + pa.rows));
    if (small)
        hipLaunchKernelGGL(prepare<0>, grid, dim3(kThreads), lds, st, pa);
    else if (four)
        hipLaunchKernelGGL(prepare<4>, grid, dim3(kThreads * 4), 0, st, pa);
    else
        hipLaunchKernelGGL(prepare<1>, grid, dim3(kThreads), 0, st, pa);
    Q8T_LAUNCH_CHECK();

    // 3. one launch over all classes (the kernel picks its class from the tile index)
    Geo g;
    g.N = d->N;
    g.IH = p.IH;
    g.IW = p.IW;
    g.Cp = p.Cp;
    g.red = p.red;
    g.OC = p.oc;
    g.OCp = p.OCp;
    g.OHf = p.OHf;
    g.OWf = p.OWf;
    g.ish = g.isw = which == 0 ? stv : 1;
    g.osh = g.osw = which == 0 ? 1 : stv;
    g.OH = g.OW = g.M = g.T = g.oph = g.opw = 0;   // per class, read by the kernel from the class table
    g.vec = q8t_aligned(out_f, 16) && q8t_aligned(out_acc, 16);
    g.ncls = ncls;
    g.fill = fill ? 1 : 0;
    // stride 2 with an even result width: the classes (ph, 0) and (ph, 1) share their positions and are
    // computed by one workgroup, which writes their interleaved results as pairs
    if (which == 1 && stv == 2 && !fill && p.OWf % 2 == 0 && cg.v[0][2] > 0) {
        const int pairM = cg.v[0][2];   // class (0, 0) is the larger row parity
#define Q8T_GOP(CFG)                                                                                                 \
    {                                                                                                                \
        static Q8tLdsOptIn optin;                                                                                    \
        if (conv_pair_lds_bytes<CFG>() > 65536 && q8t_allow_lds(optin, (const void *)igemm_nhwc_pair<CFG>, conv_pair_lds_bytes<CFG>()) != Q8T_OK)      \
            return Q8T_ERR_HIP;                                                                                      \
        g.mtiles = (pairM + CFG::BM - 1) / CFG::BM;                                                                  \
        const int64_t tiles = (int64_t)g.mtiles * 2 * (p.OCp / CFG::BN);                                              \
        hipLaunchKernelGGL(igemm_nhwc_pair<CFG>, q8t_gemm::xcd_rows(tiles), dim3(CFG::THREADS),                \
                           conv_pair_lds_bytes<CFG>(), st, xn, wt, colsum, qa, qb, g, tapoff, clsinfo, out_f, \
                           (int32_t *)out_acc);                                                                      \
    }
        if (wide_tiles(pairM, 2, p.OCp)) Q8T_GOP(q8t_gemm::Dma<128>)
        else Q8T_GOP(q8t_gemm::Dma<64>)
#undef Q8T_GOP
        Q8T_LAUNCH_CHECK();
        return Q8T_OK;
    }
#define Q8T_GO(CFG)                                                                                                  \
    {                                                                                                                \
        static Q8tLdsOptIn optin;                                                                                    \
        if (conv_lds_bytes<CFG>() > 65536 && q8t_allow_lds(optin, (const void *)igemm_nhwc<CFG>, conv_lds_bytes<CFG>()) != Q8T_OK)      \
            return Q8T_ERR_HIP;                                                                                      \
        g.mtiles = (maxM + CFG::BM - 1) / CFG::BM;                                                                   \
        const int64_t tiles = (int64_t)g.mtiles * ncls * (p.OCp / CFG::BN);                                         \
        if (tiles > 0)                                                                                               \
            hipLaunchKernelGGL(igemm_nhwc<CFG>, q8t_gemm::xcd_rows(tiles), dim3(CFG::THREADS),                 \
                               conv_lds_bytes<CFG>(), st, xn, wt, colsum, qa, qb, g, tapoff, clsinfo, out_f, \
                               (int32_t *)out_acc, bnp);                                                             \
    }
    if (wide_tiles(maxM, ncls, p.OCp)) Q8T_GO(q8t_gemm::Dma<128>)
    else Q8T_GO(q8t_gemm::Dma<64>)
#undef Q8T_GO
    Q8T_LAUNCH_CHECK();
    if (bnp)   // forward: one class, every row tile wrote its partial
        return q8t_conv_stats_finalize(bnp, p.oc, g.mtiles, g.mtiles, (double)maxM, qa, qb, bn_stats, st);
    return Q8T_OK;
}
