// Weight pre-pass of the specialised forward / layer-gradient kernels: the filter in the order their MFMA operands are
// read, plus the sum of every output channel's codes (the zero-point correction of Section 4's products).  The bodies
// live here so that one kernel can serve a single layer (conv_fast.hip, conv_wide.hip) or the filters of a whole
// network in one launch (repack_multi.hip).
#pragma once
#include "q8t_common.h"

constexpr int kRepackThreads = 512;
constexpr int kRepackCols = 16;    // output channels per workgroup
constexpr int kRepackChan = 256;   // reduction channels per round
constexpr int kRepackTaps = 9;     // at most
constexpr int kRepackRed = kRepackThreads / 64 * 16;
constexpr int kRepackLds = kRepackChan * (kRepackCols * kRepackTaps + 4);   // bytes; the larger of the two row forms below

// Layouts:
// TILE64, 64-column register-tile kernel (conv_fast.hip):
//   out[(oc/64)][cc][tap][oc%64][ch%64] = W'(oc, ch, tap);  forward: W'(oc,ch,r,s) = W[oc][ch][r][s];
//   layer gradient: W'(oc,ch,r,s) = W[ch][oc][R-1-r][S-1-s]  (oc = input channel of the layer).
// WIDE, wide-tile kernel (conv_wide.hip, 3x3), BN = 256 or 128 columns per block: block (oc / BN, chunk, tap) of BN x 64 bytes =
//   [32-column tile = oc % BN / 32][K half = ch % 64 / 32][lane = (ch % 32 / 16) * 32 + oc % 32][16 bytes = ch % 16]: every
//   MFMA operand of a wavefront is one 16-byte load per lane, 1 KB contiguous per instruction.
// colsum[oc] = sum of W'(oc,.,.).  Output and reduction channels are multiples of 64, at most kRepackTaps taps.
//
// One workgroup of kRepackThreads per 16 output channels, red: kRepackRed ints, lds: kRepackLds bytes, 4-byte aligned.  The filter
// comes in runs that lie together (an output channel's taps of all channels forward, a reduction channel's taps of 16 output
// channels backward), 16 bytes a load, and is picked apart in LDS: byte loads from memory, one line for each in the layer
// gradient, took 56 us for the filters of a ResNet-18 in both directions.  A filter on its own is a few workgroups, each bound by the
// latency of its loads and LDS reads: 512 threads (of 256, or of 1024), the next round's loads in flight across the LDS barriers and
// constant distances in LDS.  us a launch, back to back, 256 threads without these / now: 512 -> 512 3x3 10.9 / 6.7, 256 -> 256
// 6.25 / 4.1, 64 -> 64 3.7 / 2.9, 1x1 3.0 / 2.1; whole forward calls, byte loads / 256 threads / now: 512 -> 512 @7 batch 256 65.0 / 68.3 /
// 65.8, 256 -> 256 @14 44.6 / 47.9 / 45.2, 64 -> 64 @56 batch 8 11.3 / 11.0 / 10.2, 512 -> 64 1x1 @8 11.9 / 13.6 / 11.8.
template <int taps, bool dgrad>
__device__ __forceinline__ void q8t_repack_taps(const int8_t *__restrict__ w, int Kf, int Cf, int wide_bn,
                                                int8_t *__restrict__ out, int *__restrict__ colsum, int oc0, uint8_t *lds, int *red)
{
    const int CHN = dgrad ? Kf : Cf, CC = CHN / 64, tid = threadIdx.x;
    const int oc = oc0 + (tid & 15);   // of the thread's pieces
    int sum = 0;
    constexpr int U = (taps * kRepackChan + kRepackThreads - 1) / kRepackThreads;
    uint4 v[U];
    // rows in LDS: forward [output channel][channels * taps], layer gradient [reduction channel][16 * taps], `run` pieces each; 4 bytes
    // between them keep the rows of neighbouring output channels on different banks
    auto load = [&](int ch0) {
        const int pieces = taps * min(kRepackChan, CHN - ch0), run = dgrad ? taps : pieces / 16;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = min(tid + u * kRepackThreads, pieces - 1), row = p / run, at = p - row * run;
            const size_t first = dgrad ? ((size_t)(ch0 + row) * Cf + oc0) * taps : ((size_t)(oc0 + row) * Cf + ch0) * taps;
            __builtin_memcpy(&v[u], w + first + at * 16, 16);
        }
    };
    load(0);
    for (int ch0 = 0; ch0 < CHN; ch0 += kRepackChan) {
        const int pieces = taps * min(kRepackChan, CHN - ch0), run = dgrad ? taps : pieces / 16, pitch = run * 16 + 4;
        if (ch0) q8t_lds_barrier();   // the previous round's pieces are out
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = tid + u * kRepackThreads, row = p / run, at = p - row * run;
            if (p < pieces) {
                uint32_t *d = reinterpret_cast<uint32_t *>(lds + row * pitch + at * 16);
                d[0] = v[u].x;
                d[1] = v[u].y;
                d[2] = v[u].z;
                d[3] = v[u].w;
            }
        }
        if (ch0 + kRepackChan < CHN) load(ch0 + kRepackChan);
        q8t_lds_barrier();
        for (int p = tid; p < pieces; p += kRepackThreads) {
            const int e = p >> 4, tap = e % taps, c16 = e / taps;   // 16 reduction channels of one tap
            const uint8_t *src = dgrad ? lds + c16 * 16 * pitch + (tid & 15) * taps + (taps - 1 - tap)
                                       : lds + (tid & 15) * pitch + c16 * 16 * taps + tap;
            const int step = dgrad ? pitch : taps;
            uint32_t pk[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                pk[d] = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) pk[d] |= (uint32_t)src[(4 * d + i) * step] << (8 * i);
                sum = __builtin_amdgcn_sdot4((int)pk[d], 0x01010101, sum, false);
            }
            const int ch = ch0 + c16 * 16, cc = ch / 64, c64 = ch % 64;
            size_t o;
            if (wide_bn) {
                const int ob = oc % wide_bn;
                o = (((size_t)(oc / wide_bn) * CC + cc) * taps + tap) * (wide_bn * 64) + (ob / 32 * 2 + c64 / 32) * 1024 +
                    ((c64 % 32) / 16 * 32 + oc % 32) * 16;
            } else {
                o = ((((size_t)(oc / 64) * CC + cc) * taps + tap) * 64 + oc % 64) * 64 + c64;
            }
            *reinterpret_cast<uint4 *>(out + o) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        }
    }
    sum += __shfl_xor(sum, 16, Q8T_WAVE);
    sum += __shfl_xor(sum, 32, Q8T_WAVE);
    if ((tid & 63) < 16) red[(tid >> 6) * 16 + tid % 16] = sum;
    __syncthreads();
    if (tid < 16) {
        int t = 0;
#pragma unroll
        for (int i = 0; i < kRepackThreads / 64; ++i) t += red[i * 16 + tid];
        colsum[oc0 + tid] = t;
    }
}

// taps: 9 or 1
__device__ __forceinline__ void q8t_repack(const int8_t *__restrict__ w, int Kf, int Cf, int taps, int dgrad, int wide_bn,
                                           int8_t *__restrict__ out, int *__restrict__ colsum, int oc0, uint8_t *lds, int *red)
{
    if (taps == 1 && dgrad) q8t_repack_taps<1, true>(w, Kf, Cf, wide_bn, out, colsum, oc0, lds, red);
    else if (taps == 1) q8t_repack_taps<1, false>(w, Kf, Cf, wide_bn, out, colsum, oc0, lds, red);
    else if (dgrad) q8t_repack_taps<kRepackTaps, true>(w, Kf, Cf, wide_bn, out, colsum, oc0, lds, red);
    else q8t_repack_taps<kRepackTaps, false>(w, Kf, Cf, wide_bn, out, colsum, oc0, lds, red);
}

// Filters packed ahead of the products (q8t_qconv_pack): which layout a (shape, product) pair takes
enum { Q8T_PACK_NONE = 0, Q8T_PACK_TILE64 = 1, Q8T_PACK_WIDE256 = 2, Q8T_PACK_WIDE128 = 3 };

// a packed filter: [codes, K*C*R*S bytes rounded up to 256][column sums, one int per output channel of the product]
inline size_t q8t_pack_colsum_offset(const q8t_conv_desc *d) { return ((size_t)d->K * d->C * d->R * d->S + 255) & ~(size_t)255; }
inline size_t q8t_pack_bytes(int which, const q8t_conv_desc *d)
{
    return q8t_pack_colsum_offset(d) + (((size_t)(which == 0 ? d->K : d->C) * sizeof(int) + 255) & ~(size_t)255);
}

struct Q8tPackJob {
    const int8_t *w;
    int8_t *out;
    int *colsum;
    int Kf, Cf, R, S;
    int dgrad, layout;   // layout: Q8T_PACK_*
    int first_block;     // its output channels are blocks first_block .. of the launch
};
constexpr int kPackMaxJobs = 48;
// one launch for all jobs (repack_multi.hip); jobs is a host array
int q8t_pack_launch(const Q8tPackJob *jobs, int n, hipStream_t st);
