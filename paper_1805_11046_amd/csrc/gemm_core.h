// Main loops of the int8 MFMA GEMM kernels: through registers (wgrad_gemm.hip), and copied to LDS (conv_nhwc.hip, below).
//
// Through registers, three tile configurations (rows x columns of the workgroup tile, K-step 64):
//   Big    256 x 256, 8 wavefronts of 128 x 64   (one workgroup per compute unit)
//   Mid    128 x 128, 4 wavefronts of  64 x 64   (three workgroups per compute unit)
//   Small  128 x  64, 4 wavefronts of  32 x 64
// Per K-step a wavefront of the Big tile reads 12 operand fragments from LDS for 32 MFMAs, of the
// Mid tile 8 for 16: the Big tile halves the LDS and global traffic per MFMA and is what the
// MFMA-bound shapes use.
//
// LDS holds rows of 64 bytes without padding; the 16-byte chunk q of row r sits at chunk
// q ^ swz(r), which keeps the column-wise fragment reads free of bank conflicts (the row-wise
// staging stores are insensitive to the permutation).  LDS is double-buffered with one barrier per step.  The barrier orders
// LDS traffic only (q8t_lds_barrier), so the global loads of the next steps stay in flight across
// it: two named register sets hold the tiles of steps s+1 and s+2 while step s is multiplied.
// The loop body is straight-line code (no branch around a load or a store), which lets the
// compiler's wait-count bookkeeping keep the younger loads in flight; the step count is rounded
// up to an even number and the surplus step multiplies staged zeros.
//
// The kernel supplies an `Ops` object:
//   type R                             Regs, or a struct that starts with its members
//   void load(R &r, bool valid)        issue the global loads of the next K-step: a0 / a1 = chunk q of
//                                      tile rows ar and ar + RP, b0 / b1 likewise for the columns
//                                      (valid == false: any readable address, no advance)
//   void prepare(R &r, bool valid)     called right before the registers go to LDS: transform them
//                                      in place (byte-plane split, byte sums); with !valid the B
//                                      registers must become zero (and A too if sums are kept)
// with ar = tid >> 2, q = tid & 3, RP = threads / 4.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "q8t_common.h"

namespace q8t_gemm {

typedef int v4i __attribute__((ext_vector_type(4)));

// Workgroups are handed to the 8 XCDs (each with its own L2) round-robin by linear index.  The
// kernels are launched on a grid of 8*ceil(total/8) workgroups and run logical tile
// xcd_logical(blockIdx.x, total): consecutive logical tiles, which share an operand tile, then
// execute back to back on one XCD and find it in that XCD's L2.  A result >= total means "exit".
__device__ __forceinline__ int xcd_logical(int linear, int total)
{
    const int per = (total + 7) >> 3;
    return (linear & 7) * per + (linear >> 3);
}
inline unsigned xcd_grid(int64_t total) { return (unsigned)(((total + 7) >> 3) << 3); }
// Where that may be more workgroups than one dimension of a launch holds (fewer than 2^32 threads, 2^22 workgroups of 1024): rows
// of 2^kRowBits of them, of which the kernel runs tile xcd_logical(total).
constexpr int kRowBits = 21;
__device__ __forceinline__ int xcd_logical(int total)
{
    const int linear = (int)(blockIdx.y << kRowBits | blockIdx.x);
    return linear >> 3 < (total + 7) >> 3 ? xcd_logical(linear, total) : total;   // the last row is not full
}
inline dim3 xcd_rows(int64_t total)
{
    const int64_t n = ((total + 7) >> 3) << 3, row = (int64_t)1 << kRowBits;
    return n <= row ? dim3((unsigned)n) : dim3((unsigned)row, (unsigned)((n + row - 1) / row));
}

struct Regs {
    uint4 a0, a1, b0, b1;
};

__device__ __forceinline__ uint4 sel16(bool c, const uint4 &v)
{
    return make_uint4(c ? v.x : 0u, c ? v.y : 0u, c ? v.z : 0u, c ? v.w : 0u);
}

// Chunk permutation of an LDS row; depends on bits 1..2 of the row only, so rows 64 or 128 apart
// share it.  A 16-byte-per-lane LDS read is served in four phases of 16 lanes that are not
// consecutive lanes (measured on gfx950: lanes {0-3, 12-15, 20-23, 24-27} go together, and so on),
// so a fragment read (lane -> row lane % 16, chunk lane / 16) meets rows {0-3, 12-15} of one chunk
// with rows 4-11 of the next in one phase.  With this permutation those 16 accesses fall into 16
// different 16-byte bank groups: 207 bytes / clock / CU measured against 122 for the unpermuted
// layout, for an 80-byte row pitch or for permutations built for consecutive lanes.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 3; }

template <int BM_, int BN_>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_;
    static constexpr int THREADS = BM == 256 ? 512 : 256;
    static constexpr int RP = THREADS / 4;                      // rows staged per pass
    static constexpr int MT = BM == 256 ? 8 : (BN == 128 ? 4 : 2);
    static constexpr int NT = 4;
    static constexpr int NB = BN / RP;                          // column passes (1 or 2)
    static constexpr int LDS_BYTES = 2 * (BM + BN) * 64;
    static constexpr int MINB = BM == 256 ? 1 : 3;              // workgroups per compute unit aimed at
    __device__ static __forceinline__ int rowbase(int wave)
    {
        return BM == 256 ? (wave & 1) * 128 : (BN == 128 ? (wave & 1) * 64 : wave * 32);
    }
    __device__ static __forceinline__ int colbase(int wave) { return BN == 64 ? 0 : (wave >> 1) * 64; }
};
typedef Cfg<256, 256> Big;
typedef Cfg<128, 128> Mid;
typedef Cfg<128, 64> Small;

template <class C>
__device__ __forceinline__ void compute_step(const int8_t *__restrict__ sa, const int8_t *__restrict__ sb, int rowbase,
                                             int colbase, int l16, int kb, v4i (&acc)[C::MT][C::NT])
{
    v4i bf[C::NT];
#pragma unroll
    for (int nt = 0; nt < C::NT; ++nt) {
        const int row = colbase + nt * 16 + l16;
        bf[nt] = *reinterpret_cast<const v4i *>(sb + row * 64 + ((kb ^ swz(row)) * 16));
    }
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) {
        const int row = rowbase + mt * 16 + l16;
        const v4i af = *reinterpret_cast<const v4i *>(sa + row * 64 + ((kb ^ swz(row)) * 16));
#pragma unroll
        for (int nt = 0; nt < C::NT; ++nt)
            acc[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af, bf[nt], acc[mt][nt], 0, 0, 0);
    }
}

// sA: 2 * BM * 64 bytes, sB: 2 * BN * 64 bytes; tid: thread among the C::THREADS of a tile (a workgroup may hold several
// groups of them, which meet at the same barriers: as many steps in each)
template <class C, class Ops>
__device__ __forceinline__ void pipeline(Ops &ops, int steps, int8_t *__restrict__ sA, int8_t *__restrict__ sB,
                                         v4i (&acc)[C::MT][C::NT], int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, kb = lane >> 4;
    const int rowbase = C::rowbase(wave), colbase = C::colbase(wave);
    const int ar = tid >> 2;
    const int so = ar * 64 + (((tid & 3) ^ swz(ar)) * 16);   // LDS offset of the thread's chunk in row ar
    if (steps <= 0) return;
    typedef typename Ops::R R;
    R q0 = {}, q1 = {};
#define Q8T_GEMM_STORE(REGS, BUF, VALID)                                                \
    {                                                                                   \
        R t_ = REGS;                                                                    \
        ops.prepare(t_, VALID);                                                         \
        int8_t *a_ = sA + (BUF)*C::BM * 64 + so, *b_ = sB + (BUF)*C::BN * 64 + so;      \
        *reinterpret_cast<uint4 *>(a_) = t_.a0;                                         \
        *reinterpret_cast<uint4 *>(a_ + C::RP * 64) = t_.a1;                            \
        *reinterpret_cast<uint4 *>(b_) = t_.b0;                                         \
        if (C::NB == 2) *reinterpret_cast<uint4 *>(b_ + C::RP * 64) = t_.b1;            \
    }
    // one step: MFMAs on buffer S&1 while tile S+1 goes from registers to the other buffer and the
    // loads of tile S+3 are issued; everything between two barriers is one scheduling region
#define Q8T_GEMM_STEP(REGS, S)                                                          \
    {                                                                                   \
        const int buf = (S)&1;                                                          \
        compute_step<C>(sA + buf * C::BM * 64, sB + buf * C::BN * 64, rowbase, colbase, l16, kb, acc); \
        Q8T_GEMM_STORE(REGS, buf ^ 1, (S) + 1 < steps)                                  \
        ops.load(REGS, (S) + 3 < steps);                                                \
        q8t_lds_barrier();                                                              \
    }
    ops.load(q0, true);
    ops.load(q1, 1 < steps);
    Q8T_GEMM_STORE(q0, 0, true)
    ops.load(q0, 2 < steps);
    q8t_lds_barrier();
    for (int s = 0; s < steps; s += 2) {
        Q8T_GEMM_STEP(q1, s)
        Q8T_GEMM_STEP(q0, s + 1)
    }
#undef Q8T_GEMM_STEP
#undef Q8T_GEMM_STORE
}

// ---- tiles that go to LDS without registers ----------------------------------------------------------------------
// 16 bytes per lane from memory to `lds` + 16 * lane (`lds` uniform in the wavefront).  Nothing is returned to registers; the
// wavefront's vmcnt counts the transfer.  The LDS address goes through m0, a register that the compiler reserves for such uses and
// warns about; it is named as overwritten so that no value of its own is expected there afterwards.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy16_to_lds(const int8_t *g, int8_t *lds)
{
    const uint32_t o = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) int8_t *)lds);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(o), "v"(g) : "memory", "m0");
}
#pragma clang diagnostic pop

// 128 x 128 (eight wavefronts of 64 x 32) or 128 x 64 (of 32 x 32), K-steps of 128 in two buffers, two workgroups per compute
// unit.  An operand tile is LDS rows of 128 bytes, eight 16-byte pieces each, which a copy writes as 64 lanes x 16 bytes in a
// row; so the permutation that keeps the fragment reads free of bank conflicts is applied to the addresses in memory: piece s
// of LDS row r holds piece s ^ perm(r) of the step.
template <int BN_>
struct Dma {
    static constexpr int BM = 128, BN = BN_, THREADS = 512, DK = 128;
    static constexpr int WR = BN == 128 ? 2 : 4, MT = 8 / WR, NT = 2;
    static constexpr int NB = BN / 64;                          // pieces of the B tile a thread copies per step (A: 2)
    static constexpr int BUF = (BM + BN) * DK, LDS_BYTES = 2 * BUF;
    static constexpr int MINB = 4;                              // wavefronts per SIMD
    static_assert(8 / WR == MT, "the wavefronts that share rows take a row tile's sums each");
    // first row of the wavefront's row tile i: a wavefront goes round its row tiles from the one whose sums it takes
    __device__ static __forceinline__ int row(int wave, int i) { return ((wave % WR) * MT + ((i + wave / WR) & (MT - 1))) * 16; }
    __device__ static __forceinline__ int colbase(int wave) { return (wave / WR) * 32; }
    __device__ static __forceinline__ int perm(int r) { return (r >> 1) & 7; }
};

// The steps of a tile.  Ops: void issue(int8_t *buf), which copies the thread's pieces of the next step (the first 64 of its reduction
// indices only, where no more are left) and moves on; the kernel has called it once, for buffer 0.  halves: the reduction in units of 64.
// rsum: sums over the reduction of the four rows row(wave, 0) + 4 * (lane / 16) .., in every lane of the 16.  They are products with
// ones: an eighth (a quarter) more products, where sums of the operand bytes in the vector unit cost more.
template <class C, bool TIGHT, class Ops>
__device__ __forceinline__ void dma_pipeline(Ops &ops, int halves, int8_t *__restrict__ smem, v4i (&acc)[C::MT][C::NT],
                                             v4i &rsum, int tid)
{
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kb = lane >> 4;
    const int rb = C::colbase(wave) + l16;
    const v4i ones = (v4i){0x01010101, 0x01010101, 0x01010101, 0x01010101};
    rsum = (v4i){0, 0, 0, 0};
    constexpr int H1 = TIGHT ? 0 : 1;   // fragments of the second half
    v4i af[1 + H1][C::MT], bf[1 + H1][C::NT];
    auto read = [&](const int8_t *a, int h) {
#pragma unroll
        for (int j = 0; j < C::NT; ++j) {
            const int r = rb + j * 16;
            bf[h * H1][j] = *reinterpret_cast<const v4i *>(a + C::BM * C::DK + r * C::DK + (((h * 4 + kb) ^ C::perm(r)) * 16));
        }
#pragma unroll
        for (int i = 0; i < C::MT; ++i) {
            const int r = C::row(wave, i) + l16;
            af[h * H1][i] = *reinterpret_cast<const v4i *>(a + r * C::DK + (((h * 4 + kb) ^ C::perm(r)) * 16));
        }
    };
    auto multiply = [&](int h) {
#pragma unroll
        for (int i = 0; i < C::MT; ++i)
#pragma unroll
            for (int j = 0; j < C::NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[h * H1][i], bf[h * H1][j], acc[i][j], 0, 0, 0);
        rsum = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[h * H1][0], ones, rsum, 0, 0, 0);
    };
    for (int s = 0; 2 * s < halves; ++s) {
        int8_t *cur = smem + (s & 1) * C::BUF, *nxt = smem + ((s & 1) ^ 1) * C::BUF;
        // the tiles of this step are there, and every wavefront is past its reads of the other buffer
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (2 * s + 2 < halves) ops.issue(nxt);
        read(cur, 0);
        if (TIGHT) {
            multiply(0);
            if (2 * s + 1 < halves) {
                read(cur, 1);
                multiply(1);
            }
        } else if (2 * s + 1 < halves) {
            read(cur, 1);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);   // a wavefront that multiplies goes before the ones that read
            multiply(0);
            multiply(1);
        } else {
            __builtin_amdgcn_s_setprio(1);
            multiply(0);
        }
        __builtin_amdgcn_s_setprio(0);
    }
}

}  // namespace q8t_gemm
