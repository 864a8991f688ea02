// Weight pre-pass of the specialised forward / layer-gradient kernels: the filter in the order their MFMA operands are
// read, plus the sum of every output channel's codes (the zero-point correction of Section 4's products).  The bodies
// live here so that one kernel can serve a single layer (conv_fast.hip, conv_wide.hip) or the filters of a whole
// network in one launch (repack_multi.hip).
#pragma once
#include "q8t_common.h"

constexpr int kRepackThreads = 256;
constexpr int kRepackCols = 16;    // output channels per workgroup
constexpr int kRepackChan = 256;   // reduction channels per round
constexpr int kRepackTaps = 9;     // at most
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
// One workgroup of kRepackThreads per 16 output channels, red: 4 * 16 ints, lds: kRepackLds bytes, 4-byte aligned.  The filter
// comes in runs that lie together (an output channel's taps of all channels forward, a reduction channel's taps of 16 output
// channels backward), 16 bytes a load, and is picked apart in LDS: byte loads from memory, one line for each in the layer
// gradient, took 9 us for 512 -> 512 3x3 and 56 for the filters of a ResNet-18 in both directions; now 5 and 23.
__device__ __forceinline__ void q8t_repack(const int8_t *__restrict__ w, int Kf, int Cf, int taps, int dgrad, int wide_bn,
                                           int8_t *__restrict__ out, int *__restrict__ colsum, int oc0, uint8_t *lds, int *red)
{
    const int CHN = dgrad ? Kf : Cf, CC = CHN / 64, tid = threadIdx.x;
    const int oc = oc0 + (tid & 15);   // of the thread's pieces
    int sum = 0;
    for (int ch0 = 0; ch0 < CHN; ch0 += kRepackChan) {
        const int nch = min(kRepackChan, CHN - ch0), pieces = taps * nch;
        // rows in LDS: forward [output channel][nch * taps], layer gradient [reduction channel][16 * taps]; 4 bytes between them
        // keep the rows of neighbouring output channels on different banks
        const int run = dgrad ? taps : pieces / 16, pitch = run * 16 + 4;
        uint4 v[kRepackTaps];
#pragma unroll
        for (int u = 0; u < kRepackTaps; ++u) {
            if (u == 1 && pieces <= kRepackThreads) break;   // 1x1: one piece a thread
            const int p = min(tid + u * kRepackThreads, pieces - 1), row = p / run, at = p - row * run;
            const size_t first = dgrad ? ((size_t)(ch0 + row) * Cf + oc0) * taps : ((size_t)(oc0 + row) * Cf + ch0) * taps;
            __builtin_memcpy(&v[u], w + first + at * 16, 16);
        }
        if (ch0) __syncthreads();   // the previous round's pieces are out
#pragma unroll
        for (int u = 0; u < kRepackTaps; ++u) {
            const int p = tid + u * kRepackThreads, row = p / run, at = p - row * run;
            if (p < pieces) {
                uint32_t *d = reinterpret_cast<uint32_t *>(lds + row * pitch + at * 16);
                d[0] = v[u].x;
                d[1] = v[u].y;
                d[2] = v[u].z;
                d[3] = v[u].w;
            }
        }
        __syncthreads();
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
    if (tid < 16) colsum[oc0 + tid] = red[tid] + red[16 + tid] + red[32 + tid] + red[48 + tid];
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
