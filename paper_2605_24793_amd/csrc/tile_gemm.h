// The arbitration head's first layer over every decision slot in LDS tiles (the
// pre-activations U = H W1^T of Section 3.3's z = w2 . relu(W1 h + b1) + b2; bf16 heads):
// in a chain step's reduction launch, beside the units that stream the logits, and on its
// own in the second phase of a split step.
//
// The hidden states do not depend on the reduction, and a reduction that waits for HBM
// leaves the matrix cores and most of L2 idle, so scoring every slot beside it costs less
// than scoring the mismatches after it.  Two things decide what it costs: the registers
// and LDS of this code are those of every workgroup of the launch (64 VGPRs and 16 KB keep
// the reduction's eight waves per SIMD: with 32 KB, five, the reduction of 64 x K=7 took 59
// us instead of 51), and these workgroups hold places that would otherwise stream, so
// they are few (at most one per CU) and each runs long.
//
// A workgroup of four waves takes a 64 x 64 tile of U over part of d: 64-byte k-steps of 64
// gathered hidden rows and 64 W1 rows go straight into an LDS ring, and each wave
// accumulates 32 x 32 (v_mfma_f32_32x32x16_bf16).  d is cut into a.kslices slices, each summed
// by itself; a workgroup runs a.kgroup of them and adds their sums in order, and where it runs
// one the second layer adds them in the same groups (HeadArgs::zgroup).  So z is the same bits
// in both forms.  The slices are as many as the tiled GEMM and the slot GEMM take at the same
// sizes (8, 16 or 32): with 8 throughout, the relative error of z grew where those take more
// (120 slots, 4096 -> 256: 1.48e-7 -> 1.73e-7, now 1.36e-7).  Workgroups of one slice group stay on the same
// XCDs (the groups, 2, 4 or 8 of them, are dealt with the workgroups), whose L2 then reads
// that part of the operands.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "head_z.h"
#include "launch.h"
#include "mfma.h"

namespace cospec {
namespace tilegemm {

constexpr int kTile = kHeadSmallTile;         // slots and columns of a workgroup's tile
constexpr int kRowBytes = 64;                 // bytes of k per row and stage
constexpr int kOperand = kTile * kRowBytes;   // 4 KB: a stage's slots; its columns follow
constexpr int kBeside = 2;                    // ring stages beside the reduction (16 KB)
constexpr int kAlone = 4;                     // ... and on its own
constexpr int lds_bytes(int stages) { return stages * 2 * kOperand; }

typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((address_space(3))) const char lds_cchar;

__host__ __device__ inline int64_t blocks(const HeadArgs &a) {
    return (a.m_cap + kTile - 1) / kTile * ((a.h + kTile - 1) / kTile) * a.ksplit;
}

// Loads 16 bytes per lane from global memory straight into LDS, lane l's at byte lds + 16 l.
// Assembly, so that the compiler places no wait for it before the LDS reads of other stages;
// the waits below order them.  M0 is declared clobbered; nothing else here uses it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void load_lds16(const void *g, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(g) : "memory", "m0");
}
#pragma clang diagnostic pop

// Waits until at most N vector-memory operations of this wave are outstanding.
template <int N> __device__ inline void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Workgroup w of blocks(a).  lds: lds_bytes(STAGES) of LDS; zero: sixteen zero bytes in device
// memory, loaded for the pieces past the end of d.
template <int STAGES>
__device__ inline void run(const HeadArgs &a, int w, char *lds, const u32x4 *zero) {
    static_assert(STAGES >= 2 && STAGES <= 4, "the stage waits");
    constexpr int EB = 2, VE = 8, KE = kRowBytes / EB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m_cap = static_cast<int>(a.m_cap);
    const int row_tiles = (m_cap + kTile - 1) / kTile;
    const int ks = w % a.ksplit, t = w / a.ksplit;
    const int s0 = t % row_tiles * kTile, n0 = t / row_tiles * kTile;
    // a slice is whole stages (whole 128-byte pieces left the workgroups of 5120 elements in 32
    // slices 768 elements each, the last ones none: two trees of 38 nodes 26.1 us instead of
    // 24.8)
    const int kslice = ((a.d + a.kslices - 1) / a.kslices + KE - 1) / KE * KE;
    const int k0 = ks * a.kgroup * kslice, k1 = min(a.d, k0 + a.kgroup * kslice);
    const int nst = k1 > k0 ? (k1 - k0 + KE - 1) / KE : 0, slice_st = kslice / KE;

    // loader: this lane brings the 16 bytes at 16 * lane of the wave's 1 KB of each operand,
    // i.e. row 16 * wave + lane / 4, unit lane % 4, which holds k-vector unit ^ swizzle(row)
    // (rows 4 apart differ, so that 16 rows read at one column hit distinct LDS banks).  A
    // slot past the last reads the last slot's row and an invalid hidden row row 0: never
    // stored, and z = NaN in the second layer.
    const int lrow = 16 * wave + (lane >> 2), lvec = (lane & 3) ^ ((lrow >> 2) & 3);
    int64_t id = headz::mapped_row(a, min(s0 + lrow, m_cap - 1));
    if (id < 0 || id >= a.n_rows) id = 0;
    const char *ga = static_cast<const char *>(a.hidden) + id * static_cast<int64_t>(a.d) * EB;
    const char *gb = static_cast<const char *>(a.w1) + static_cast<int64_t>(min(n0 + lrow, a.h - 1)) * a.d * EB;
    const uint32_t base = __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_cchar *)lds)) + wave * 1024);
    auto issue = [&](int st) {
        const int e = k0 + st * KE + lvec * VE;   // d is a multiple of VE
        const bool in = e < k1;
        const uint32_t slot = base + st % STAGES * (2 * kOperand);
        load_lds16(in ? static_cast<const void *>(ga + static_cast<int64_t>(e) * EB) : zero, slot);
        load_lds16(in ? static_cast<const void *>(gb + static_cast<int64_t>(e) * EB) : zero, slot + kOperand);
    };

    // products: wave (wave / 2, wave % 2) takes 32 slots x 32 columns
    const int l32 = lane & 31, g = lane >> 5;
    const int ra = 32 * (wave >> 1) + l32, rb = 32 * (wave & 1) + l32;
    const int oa = ra * kRowBytes, ob = kOperand + rb * kRowBytes;
    const int sa = (ra >> 2) & 3, sb = (rb >> 2) & 3;
    floatx16 acc, sum;
#pragma unroll
    for (int i = 0; i < 16; ++i) { acc[i] = 0.f; sum[i] = 0.f; }
#pragma unroll
    for (int st = 0; st < STAGES - 1; ++st)
        if (st < nst) issue(st);
    int left = slice_st;                          // stages of the slice still to come
    for (int st = 0; st < nst; ++st) {
        // this wave's two loads of stage st are done once at most the later stages' remain
        const int later = min(STAGES - 2, nst - 1 - st);
        if (STAGES >= 4 && later >= 2) wait_vm<4>();
        else if (STAGES >= 3 && later == 1) wait_vm<2>();
        else wait_vm<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();             // landed everywhere; stage st - 1 read by all
        asm volatile("" ::: "memory");
        if (st + STAGES - 1 < nst) issue(st + STAGES - 1);
        const char *p = lds + st % STAGES * (2 * kOperand);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const u32x4 av = *reinterpret_cast<const u32x4 *>(p + oa + ((2 * s + g) ^ sa) * 16);
            const u32x4 bv = *reinterpret_cast<const u32x4 *>(p + ob + ((2 * s + g) ^ sb) * 16);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv),
                                                          acc, 0, 0, 0);
        }
        if (--left == 0 && a.kgroup > 1) {        // the slice is done: wave-uniform
            left = slice_st;
#pragma unroll
            for (int i = 0; i < 16; ++i) { sum[i] += acc[i]; acc[i] = 0.f; }
        }
    }
    // element i: slot 8 (i / 4) + 4g + i % 4 of the wave's, column l32; nontemporal stores:
    // the partials are read once, by the finish
    float *up = a.upart + static_cast<int64_t>(ks) * m_cap * a.h;
    const int n = n0 + rb;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int s = s0 + ra - l32 + 8 * (i / 4) + 4 * g + i % 4;
        if (s < m_cap && n < a.h) __builtin_nontemporal_store(sum[i] + acc[i], &up[static_cast<int64_t>(s) * a.h + n]);
    }
}

}  // namespace tilegemm
}  // namespace cospec
