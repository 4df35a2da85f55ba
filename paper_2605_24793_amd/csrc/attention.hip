// The arbitrator's hybrid attention (Section 3.3).  The arbitrator reads
// q = [context, SEP, draft 1..K, SEP, candidates 1..K, SEP] (Eq. arb_input) of
// length l = l_c + 2K + 3 under a hybrid mask: context positions attend causally
// within the context; the draft/target region, read as starting at the first SEP
// (position l_c), attends to the whole context and bidirectionally within itself;
// nothing flows from the region back into the context.
//
// k_hybrid_mask writes that mask densely ([B][L][L] bytes, 1 = attend; padding
// rows attend only to themselves) for attention code that takes explicit masks.
//
// k_hybrid_attention computes softmax(q k^T * scale + mask) v for a range of query
// positions of each sequence straight from the rule (no mask in memory), with
// grouped query heads, bf16 inputs and fp32 accumulation on the matrix cores.
// Per round only the region's 2K+3 queries are new: their keys and values are
// the cached context plus the region itself.
//
// Work split (k_hybrid_attention; k_hybrid_attention_wide below takes groups of more than
// 128 rows): the query rows (position x head) that share one key/value head of
// one sequence go to one workgroup of up to 8 waves, 16 rows per wave, so each
// key and value is read once per group.  Keys and
// values stream through a ring of kStages LDS stages of kKeyBlock rows, filled
// straight from HBM by raw buffer loads into LDS (no register staging): the
// buffers end after the group's last visible row, so the hardware range check
// fills later rows with zeros.  Both tiles are stored row-major with an XOR
// swizzle of their 16- or 32-byte units so that the fragment reads below hit
// distinct LDS banks.  Each wave computes S^T = K Q^T
// (v_mfma_f32_16x16x32_bf16, A = K rows from LDS, B = its queries' columns kept
// in registers), so lane l owns query column l % 16 of S^T and keeps that query's
// running max and sum (online softmax).  P^T is packed to bf16 in the same lanes
// and O^T += V^T P^T takes its A operand (V^T) from the row-major V tile with the
// gfx950 transposing LDS read (ds_read_b64_tr_b16), leaving O^T[d][query] in the
// lane that owns the query, so rescaling needs no exchange.
//
// Few groups (small batches) leave most CUs without work, so their keys are cut into
// pieces (attn_plan): the SPLIT form writes each piece's unnormalised sums, and
// k_attention_combine merges them.  Two sequences of 16401 and 8209 positions, 8 key/value
// heads, 17 queries of 32 heads: 330 us on 16 workgroups, 32 us in pieces of 1056 keys
// (25 us of it the pieces, 4.5 us the merge; 101 MB of keys and values).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "launch.h"

namespace cospec {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kKeyBlock = 32;         // key rows per LDS stage
constexpr int kStages = 4;            // LDS ring: three stages in flight while one is used
// waves that issue the loads (a workgroup has at least 4): two measured 2% faster than
// four at 64 x 2048 context (96.5-98.6 against 99.3-100.0 us on one box), one the same
constexpr int kLoaders = 2;
constexpr int kMaxWaves = 8;          // per workgroup, 16 query rows each (register budget)
constexpr float kLog2eA = 1.4426950408889634f;

// Word 3 of a raw (unswizzled, stride 0) buffer resource: 32-bit data format.
constexpr int kRawBuffer = 0x00020000;

typedef __attribute__((address_space(3))) void lds_void;

constexpr int kNontemporal = 2;       // cache policy of the key/value loads: streamed once

// 16 bytes per lane from a raw buffer into LDS at base + 16 * lane (zeros past the
// buffer's end).  Nontemporal: each key and value is read once per round (measured at
// 64 sequences x 2048 context positions: 109 -> 98 us; a fifth key stage, an earlier
// issue of the value reads or two accumulator chains for S changed nothing more).
__device__ inline void load_lds16(__amdgpu_buffer_rsrc_t r, uint32_t off, const char *lds) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)lds, 16, static_cast<int>(off), 0, 0, kNontemporal);
}

// Waits until at most N vector-memory operations of this wave are outstanding.
template <int N> __device__ inline void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Waits until this wave has at most PER * later of its loads in flight, later <= MAXL.
template <int PER, int MAXL> __device__ inline void wait_later(int later) {
    if constexpr (MAXL > 0) {
        if (later >= MAXL) wait_vm<PER * MAXL>();
        else wait_later<PER, MAXL - 1>(later);
    } else {
        wait_vm<0>();
    }
}

// Workgroup barrier that does not wait for the stages still in flight (as the fence
// of __syncthreads would); the compiler may not move memory accesses across it.
__device__ inline void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Transposing LDS read: within each row of 16 lanes, lane j receives element j % 4 of
// the 8-byte chunks addressed by lanes 4k + j / 4, k = 0..3 (in that order).  Issued
// as inline assembly: the compiler does not know which LDS the builtin reads and
// would wait for every load into LDS still in flight before it.  The caller waits for
// the result with lds_wait().
typedef __attribute__((address_space(3))) const char lds_cchar;
__device__ inline u32x2 read_tr(const char *lds) {
    const uint32_t addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_cchar *)lds));
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(r) : "v"(addr));
    return r;
}

// Waits for this wave's LDS reads; the values passed through are only used after it.
template <int N> __device__ inline void lds_wait(u32x2 (&x)[N], u32x2 (&y)[N]) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]), "+v"(y[i]));
}

// A value that is the same in every lane, for the scalar registers (a buffer descriptor
// built from a value the compiler keeps in a vector register costs a loop per load).
__device__ inline int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// XOR swizzles of the LDS tiles (rows of RB = 2D bytes).  K: 16-byte units, so that
// 16 consecutive rows read at one column hit distinct banks; V: 32-byte units, so
// that the 8 rows of a transposing read do.
template <int RB> __device__ inline int swz_k(int row) { return RB == 256 ? (row & 15) : ((row >> 1) & 7); }
template <int RB> __device__ inline int swz_v(int row) { return RB == 256 ? (row & 7) : ((row >> 1) & 3); }

__device__ inline floatx4 mfma(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                   c, 0, 0, 0);
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// Two fp32 values -> one word of two bf16 (lo in bits 0-15), round to nearest even
// (v_cvt_pk_bf16_f32).
__device__ inline uint32_t bf16_pair(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, bf16x2{static_cast<__bf16>(lo), static_cast<__bf16>(hi)});
}

// max over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the rows of 16 lanes), in the VALU
__device__ inline float max_rows(float x) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

__device__ inline float sum_rows(float x) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// The running max of a query is only raised when a block's max exceeds it by more
// than this (log2 units), so that the accumulators are rarely rescaled; weights stay
// below 2^kLazyRescale.
constexpr float kLazyRescale = 8.0f;

__global__ __launch_bounds__(256) void k_hybrid_mask(MaskArgs a) {
    const int64_t row = blockIdx.x;                         // b * L + i
    const int b = static_cast<int>(row / a.L), i = static_cast<int>(row % a.L);
    const int lc = max(a.ctx_len[b], 0);
    const int64_t ln = static_cast<int64_t>(lc) + 2 * a.K + 3;
    uint8_t *out = a.mask + row * a.L;
    for (int j = threadIdx.x; j < a.L; j += blockDim.x) {
        bool m;
        if (i >= ln) m = j == i;
        else if (i < lc) m = j <= i;
        else m = j < ln;
        out[j] = m;
    }
}

// SPLIT: the keys of every group are cut into pieces of a.chunk rows (a multiple of
// kKeyBlock), one workgroup each, and the workgroup leaves its rows' unnormalised sums,
// running max and weight sum in the workspace for k_attention_combine.
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kMaxWaves) void k_hybrid_attention(AttnArgs a) {
    constexpr int RB = D * 2;                               // bytes per key/value row
    constexpr int SB = kKeyBlock * RB;                      // bytes of one tile per stage
    constexpr int LPW = SB / 1024 / kLoaders;               // 1 KB load instructions per tile and loader
    constexpr int DS = D / 32;                              // MFMA k-steps over d
    constexpr int DT = D / 16;                              // d tiles of the output
    static_assert(LPW >= 1 && kKeyBlock == 32, "stage shape");
    __shared__ __attribute__((aligned(16))) char s_k[kStages][SB];
    __shared__ __attribute__((aligned(16))) char s_v[kStages][SB];

    const int grp = a.by_grp.d;
    const int rows = a.n_q * grp;                           // query rows of one (sequence, kv head)
    const int wg_rows = blockDim.x / 4;                     // 16 rows per wave
    const uint32_t unit = SPLIT ? quot(a.by_splits, blockIdx.x) : blockIdx.x;
    const int split = SPLIT ? blockIdx.x - unit * a.splits : 0;
    const uint32_t bh = quot(a.by_wgs, unit);
    const int b = quot(a.by_hkv, bh);
    const int h = bh - b * a.Hkv;
    const int q0 = (unit - bh * a.by_wgs.d) * wg_rows;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, l16 = lane & 15;

    // this lane's query column; its loads wait for no other load
    const int qi = q0 + wave * 16 + l16;
    const bool qvalid = qi < rows;
    const int r = qvalid ? quot(a.by_grp, qi) : 0;
    const int hq = h * grp + (qvalid ? qi - r * grp : 0);
    u32x4 qf[DS];
    const char *qrow = static_cast<const char *>(a.q) + ((static_cast<int64_t>(b) * a.n_q + r) * a.Hq + hq) * D * 2;
#pragma unroll
    for (int s = 0; s < DS; ++s) qf[s] = *reinterpret_cast<const u32x4 *>(qrow + (32 * s + 8 * g) * 2);

    const int lc = uniform(max(a.ctx_len[b], 0));
    const int ln = static_cast<int>(min(static_cast<int64_t>(lc) + 2 * a.K + 3, static_cast<int64_t>(a.L)));
    const int qs = uniform(a.q_start[b]);
    // the last key any query of this workgroup sees
    const int r_hi = min(q0 + wg_rows, rows) - 1;
    const int p_lo = qs + static_cast<int>(quot(a.by_grp, q0));
    const int p_hi = qs + static_cast<int>(quot(a.by_grp, r_hi));
    const int kvis = p_lo >= ln ? 0 : p_hi >= lc ? ln : min(p_hi + 1, ln);   // all padding: no key
    // this workgroup's keys [kbeg, kend); a piece past the last visible key is left by
    // the whole workgroup (the combine reads only pieces that hold a visible key)
    const int kbeg = split * (SPLIT ? a.chunk : 0);
    if (SPLIT && kbeg >= kvis) return;
    const int kend = uniform(SPLIT ? min(kvis, kbeg + a.chunk) : kvis);

    const int p = qs + r;
    const bool live = qvalid && p >= 0 && p < ln;
    const int vis = p < lc ? p + 1 : ln;                   // keys [0, vis) are visible
    // the query loads complete here, not at their first use inside the key loop (where
    // the wait would also cover every key/value load issued after them)
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        asm volatile("" : "+v"(qf[s]));
        qf[s] = live ? qf[s] : u32x4{0, 0, 0, 0};
    }

    floatx4 o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) o[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    // m: running max of the scaled scores (log2 units), common to the four lanes of a
    // query column; l: this lane's share of the running sum (its keys 4g + j)
    float m = -INFINITY, l = 0.f;
    const float sc = a.scale * kLog2eA;
    // blocks that end at or below every lane's visible length need no mask
    int vis_min = vis;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) vis_min = min(vis_min, __shfl_xor(vis_min, off));

    // raw buffers over this group's keys and values, ending after row kend - 1;
    // offsets are 32-bit (L * Hkv * D * 2 < 2^32)
    const uint32_t row_b = static_cast<uint32_t>(a.Hkv) * D * 2;   // bytes between positions
    const int64_t head0 = (static_cast<int64_t>(b) * a.L * a.Hkv + h) * D * 2;
    const int nbytes = kend > 0 ? static_cast<int>((kend - 1) * row_b + RB) : 0;
    const __amdgpu_buffer_rsrc_t krs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(static_cast<const char *>(a.k) + head0), 0, nbytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t vrs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(static_cast<const char *>(a.v) + head0), 0, nbytes, kRawBuffer);

    // loader wave w, instruction q fills bytes (w * LPW + q) KB of a tile: lane l the
    // 16 bytes at 16 l of that KB, i.e. row `lrow`, physical unit `pch` of the tile,
    // which holds logical unit pch ^ swizzle(row)
    const bool loader = wave < kLoaders;
    uint32_t koff[LPW], voff[LPW];
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
        const int o16 = ((wave * LPW + q) * 1024 + lane * 16);
        const int lrow = o16 / RB, pch = (o16 % RB) / 16;
        koff[q] = lrow * row_b + (pch ^ swz_k<RB>(lrow)) * 16;
        voff[q] = lrow * row_b + (((pch >> 1) ^ swz_v<RB>(lrow)) * 2 + (pch & 1)) * 16;
    }
    const int nblk = (kend - kbeg + kKeyBlock - 1) / kKeyBlock;
    auto issue = [&](int j) {
        const uint32_t off = static_cast<uint32_t>(kbeg + j * kKeyBlock) * row_b;
        const char *lk = s_k[j % kStages] + wave * LPW * 1024;
        const char *lv = s_v[j % kStages] + wave * LPW * 1024;
#pragma unroll
        for (int q = 0; q < LPW; ++q) {
            load_lds16(krs, koff[q] + off, lk + q * 1024);
            load_lds16(vrs, voff[q] + off, lv + q * 1024);
        }
    };
    if (loader) {
#pragma unroll
        for (int j = 0; j < kStages - 1; ++j)
            if (j < nblk) issue(j);
    }

    for (int j = 0; j < nblk; ++j) {
        // this wave's loads of stage j are done once at most the later stages' remain
        wait_later<2 * LPW, kStages - 2>(min(kStages - 2, nblk - 1 - j));   // 2 LPW loads per stage
        lds_barrier();                                      // stage j landed; stage j-1 consumed
        if (loader && j + kStages - 1 < nblk) issue(j + kStages - 1);
        const char *sk = s_k[j % kStages];
        const char *sv = s_v[j % kStages];
        const int k0 = kbeg + j * kKeyBlock;

        // S^T[key][query] for the block: tile c holds keys 16c + 4g + jj in element jj
        floatx4 st[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int row = 16 * c + l16;
            u32x4 kf[DS];
#pragma unroll
            for (int s = 0; s < DS; ++s)
                kf[s] = *reinterpret_cast<const u32x4 *>(sk + row * RB + ((4 * s + g) ^ swz_k<RB>(row)) * 16);
            st[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < DS; ++s) st[c] = mfma(kf[s], qf[s], st[c]);
        }
        // online softmax over this block, for the query in this lane's column
        float bm = -INFINITY;
        if (k0 + kKeyBlock <= vis_min) {                     // wave-uniform: no key masked
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    st[c][jj] *= sc;
                    bm = fmaxf(bm, st[c][jj]);
                }
        } else {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int key = k0 + 16 * c + 4 * g + jj;
                    st[c][jj] = key < vis ? st[c][jj] * sc : -INFINITY;
                    bm = fmaxf(bm, st[c][jj]);
                }
        }
        bm = max_rows(bm);
        const bool raise = bm > m + kLazyRescale;            // always when m is still -inf
        if (__builtin_expect(__ballot(raise) != 0, 0)) {
            const float alpha = raise ? __builtin_amdgcn_exp2f(m - bm) : 1.f;   // 0 from -inf
            if (raise) m = bm;
            l *= alpha;
#pragma unroll
            for (int t = 0; t < DT; ++t) o[t] *= alpha;
        }
        // a lane whose keys so far are all masked keeps m = -inf and adds nothing
        const float mm = m == -INFINITY ? INFINITY : m;
        uint32_t pk[2][2];                                   // P^T as bf16 pairs, tile c
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float pv[4];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                pv[jj] = __builtin_amdgcn_exp2f(st[c][jj] - mm);
                l += pv[jj];
            }
            pk[c][0] = bf16_pair(pv[0], pv[1]);
            pk[c][1] = bf16_pair(pv[2], pv[3]);
        }
        // O^T[d][query] += V^T[d][keys] P^T[keys][query].  The B operand of lane
        // group g holds keys 4g + 0..3 and 16 + 4g + 0..3; the transposing reads give
        // lane (g, d) the same keys of V column d: lane 4k + c of the group addresses
        // key 4g + k (or 16 + 4g + k), values 16t + 4c .. 16t + 4c + 3.
        const u32x4 pb{pk[0][0], pk[0][1], pk[1][0], pk[1][1]};
        const int vr0 = 4 * g + (l16 >> 2), vr1 = vr0 + 16;
        const int vb = 8 * (l16 & 3);
        u32x2 lo[DT], hi[DT];
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            lo[t] = read_tr(sv + vr0 * RB + (t ^ swz_v<RB>(vr0)) * 32 + vb);
            hi[t] = read_tr(sv + vr1 * RB + (t ^ swz_v<RB>(vr1)) * 32 + vb);
        }
        lds_wait(lo, hi);
#pragma unroll
        for (int t = 0; t < DT; ++t) o[t] = mfma(u32x4{lo[t][0], lo[t][1], hi[t][0], hi[t][1]}, pb, o[t]);
    }

    l = sum_rows(l);
    if (!qvalid) return;
    if constexpr (SPLIT) {
        // nontemporal stores: read once, by the combine
        const int64_t rows_all = static_cast<int64_t>(a.B) * a.n_q * a.Hq;
        const int64_t R = split * rows_all + (static_cast<int64_t>(b) * a.n_q + r) * a.Hq + hq;
        float *po = a.part_o + R * D + 4 * g;
#pragma unroll
        for (int t = 0; t < DT; ++t) __builtin_nontemporal_store(o[t], reinterpret_cast<floatx4 *>(po + 16 * t));
        if (g == 0) a.part_ml[R] = make_float2(m, l);
        return;
    }
    // O^T tile t, element j: d = 16t + 4g + j of this lane's query
    char *orow = static_cast<char *>(a.out) + ((static_cast<int64_t>(b) * a.n_q + r) * a.Hq + hq) * D * 2;
    const float inv = live && l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int t = 0; t < DT; ++t) {
        const uint32_t w0 = bf16_pair(o[t][0] * inv, o[t][1] * inv);
        const uint32_t w1 = bf16_pair(o[t][2] * inv, o[t][3] * inv);
        *reinterpret_cast<u32x2 *>(orow + (16 * t + 4 * g) * 2) = u32x2{w0, w1};
    }
}

// ---------------------------------------------------------------- many query rows

typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) short shortx4;

constexpr int kWideKeys = 64;         // keys per LDS stage
constexpr int kWideWaves = 4;         // 32 query rows each
constexpr int kWideRows = 32 * kWideWaves;

__device__ inline floatx16 mfma32(u32x4 a, u32x4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                   c, 0, 0, 0);
}

// 16 bytes per lane from a raw buffer into LDS at byte lds + 16 * lane, lds the same in every
// lane (zeros past the buffer's end).  Written as assembly, so that the compiler, which knows nothing of these loads,
// places no wait for them before the LDS reads; the kernel's own waits order them.  M0 is
// declared clobbered and nothing else in the kernel uses it.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void load_lds16_asm(u32x4 rsrc, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(lds), "v"(off), "s"(rsrc)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

__device__ inline uint32_t lds_addr(const char *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_cchar *)p));
}

__device__ inline u32x4 raw_rsrc(const char *p, int bytes) {
    const uint64_t addr = reinterpret_cast<uint64_t>(p);
    return u32x4{static_cast<uint32_t>(uniform(static_cast<int>(addr))),
                 static_cast<uint32_t>(uniform(static_cast<int>(addr >> 32))) & 0xffffu,
                 static_cast<uint32_t>(uniform(bytes)), static_cast<uint32_t>(kRawBuffer)};
}

// The transposing LDS read of the kernel above as the builtin: every load into LDS of this
// kernel is assembly, so the compiler tracks the read like any other.
__device__ inline u32x2 read_tr_tracked(const char *lds) {
    typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)(lds_cchar *)lds));
}

// XOR swizzle of the value tiles (32-byte units): 32 lanes of a transposing read take two
// neighbouring units of each of four rows, so rows 0..3 (modulo 4) shift by pairs of units.
template <int RB> __device__ inline int swz_vw(int row) { return RB == 256 ? 2 * (row & 3) : row & 2; }

// The same attention for calls with many query rows per (sequence, key/value head), such as
// a first pass over a whole input.  There the matrix cores and the LDS bound it: sixteen
// rows per wave read every key and value from LDS twice as often as the products need.  So
// a wave takes 32 rows (32 x 32 products, D / 32 output tiles in registers), four waves
// share a two-stage ring of 64-key stages (64 KB), and two workgroups share a CU, so that
// one's softmax runs beside the other's products.  Measured, 4 sequences of 1041 to 2065
// positions, 32/8 heads, D = 128 (84 GFLOP): 200 us with 16-row waves (50 us of it on
// tiles of padding rows, which now read no key), 109-115 us here = 750 TFLOP/s, the issued
// products alone 42 us.  Also measured there: eight waves with four stages 116 us, 32-key
// stages 114 to 122, the next block's scores taken beside this block's softmax 118, three
// waves per SIMD spill.  Without the loads the same code takes 94 us, without the
// exponentials 104.
template <int D>
__global__ __launch_bounds__(64 * kWideWaves, 2) void k_hybrid_attention_wide(AttnArgs a) {
    constexpr int RB = D * 2;                               // bytes per key/value row
    constexpr int SB = kWideKeys * RB;                      // bytes of one tile per stage
    constexpr int LPW = SB / 1024 / kWideWaves;             // 1 KB load instructions per tile and wave
    constexpr int DS = D / 16;                              // MFMA k-steps over d
    constexpr int DT = D / 32;                              // d tiles of the output
    constexpr int KT = kWideKeys / 32;                      // key tiles of a stage
    __shared__ __attribute__((aligned(16))) char s_k[2][SB];   // two stages of keys
    __shared__ __attribute__((aligned(16))) char s_v[2][SB];   // ... and of values

    const int grp = a.by_grp.d;
    const int rows = a.n_q * grp;
    // Workgroups are dealt to the XCDs round-robin: with a multiple of kXcds groups
    // (a.splits = kXcds, else 1) a group's workgroups stay on one XCD, whose L2 then holds
    // its keys and values.  The last query rows come first: they see the most keys.  Group
    // by group (a.chunk = 0, by_wgs the tiles of a group), so that few groups' keys share
    // an L2 at a time; tile by tile over all groups (a.chunk = 1, by_wgs the groups of an
    // XCD) when every workgroup is resident at once.
    const bool dealt = a.splits > 1;
    const uint32_t x = dealt ? blockIdx.x % kXcds : 0, i0 = dealt ? blockIdx.x / kXcds : blockIdx.x;
    const uint32_t q0t = quot(a.by_wgs, i0), rem = i0 - q0t * a.by_wgs.d;
    const uint32_t t0 = a.chunk ? q0t : rem, lg = a.chunk ? rem : q0t;
    const uint32_t bh = lg * (dealt ? kXcds : 1) + x;
    const int b = quot(a.by_hkv, bh);
    const int h = bh - b * a.Hkv;
    const int tiles = (rows + kWideRows - 1) / kWideRows;
    const int q0 = (tiles - 1 - static_cast<int>(t0)) * kWideRows;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 5, l32 = lane & 31, l16 = lane & 15, dh = (lane >> 4) & 1;

    // this lane's query column
    const int qi = q0 + wave * 32 + l32;
    const bool qvalid = qi < rows;
    const int r = qvalid ? quot(a.by_grp, qi) : 0;
    const int hq = h * grp + (qvalid ? qi - r * grp : 0);
    u32x4 qf[DS];
    const char *qrow = static_cast<const char *>(a.q) + ((static_cast<int64_t>(b) * a.n_q + r) * a.Hq + hq) * D * 2;
#pragma unroll
    for (int s = 0; s < DS; ++s) qf[s] = *reinterpret_cast<const u32x4 *>(qrow + (16 * s + 8 * g) * 2);

    const int lc = uniform(max(a.ctx_len[b], 0));
    const int ln = static_cast<int>(min(static_cast<int64_t>(lc) + 2 * a.K + 3, static_cast<int64_t>(a.L)));
    const int qs = uniform(a.q_start[b]);
    const int r_hi = min(q0 + kWideRows, rows) - 1;
    const int p_lo = qs + static_cast<int>(quot(a.by_grp, q0));
    const int p_hi = qs + static_cast<int>(quot(a.by_grp, r_hi));
    const int kend = uniform(p_lo >= ln ? 0 : p_hi >= lc ? ln : min(p_hi + 1, ln));   // all padding: no key
    const int p = qs + r;
    const bool live = qvalid && p >= 0 && p < ln;
    const int vis = p < lc ? p + 1 : ln;                   // keys [0, vis) are visible
    // scores are taken as |scale| * (+-q) . k: the largest product is then the largest score
    const uint32_t flip = a.scale < 0.f ? 0x80008000u : 0u;
    const float sc = fmaxf(fabsf(a.scale) * kLog2eA, 1.17549435e-38f);
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        asm volatile("" : "+v"(qf[s]));
#pragma unroll
        for (int w = 0; w < 4; ++w) qf[s][w] = live ? qf[s][w] ^ flip : 0u;
    }
    int vis_min = live ? vis : INT_MAX;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) vis_min = min(vis_min, __shfl_xor(vis_min, off));

    floatx16 o[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[t][i] = 0.f;
    float m = -INFINITY, l = 0.f;

    const uint32_t row_b = static_cast<uint32_t>(a.Hkv) * D * 2;
    const int64_t head0 = (static_cast<int64_t>(b) * a.L * a.Hkv + h) * D * 2;
    const int nbytes = kend > 0 ? static_cast<int>((kend - 1) * row_b + RB) : 0;
    const u32x4 krs = raw_rsrc(static_cast<const char *>(a.k) + head0, nbytes);
    const u32x4 vrs = raw_rsrc(static_cast<const char *>(a.v) + head0, nbytes);
    uint32_t koff[LPW], voff[LPW];
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
        const int o16 = ((wave * LPW + q) * 1024 + lane * 16);
        const int lrow = o16 / RB, pch = (o16 % RB) / 16;
        koff[q] = lrow * row_b + (pch ^ swz_k<RB>(lrow)) * 16;
        voff[q] = lrow * row_b + (((pch >> 1) ^ swz_vw<RB>(lrow)) * 2 + (pch & 1)) * 16;
    }
    const int nblk = (kend + kWideKeys - 1) / kWideKeys;
    const uint32_t lds_k = uniform(lds_addr(s_k[0]) + wave * LPW * 1024);
    const uint32_t lds_v = uniform(lds_addr(s_v[0]) + wave * LPW * 1024);
    auto issue = [&](int j) {
        const uint32_t off = static_cast<uint32_t>(j * kWideKeys) * row_b, slot = (j & 1) * SB;
#pragma unroll
        for (int q = 0; q < LPW; ++q) load_lds16_asm(krs, koff[q] + off, lds_k + slot + q * 1024);
#pragma unroll
        for (int q = 0; q < LPW; ++q) load_lds16_asm(vrs, voff[q] + off, lds_v + slot + q * 1024);
    };
    // LDS addresses of this lane's fragments within a stage: the swizzles depend on the row
    // modulo 16 (keys) and 8 (values) only, so the rest is a constant offset of the read
    uint32_t ka[DS], va[DT];
#pragma unroll
    for (int s = 0; s < DS; ++s) ka[s] = l32 * RB + ((2 * s + g) ^ swz_k<RB>(l32)) * 16;
    const int vrow = 4 * g + (l16 >> 2);
#pragma unroll
    for (int t = 0; t < DT; ++t) va[t] = vrow * RB + ((2 * t + dh) ^ swz_vw<RB>(vrow)) * 32 + 8 * (l16 & 3);

    if (nblk > 0) issue(0);
    for (int j = 0; j < nblk; ++j) {
        wait_vm<0>();                                       // this wave's loads of stage j
        lds_barrier();                                      // stage j landed; stage j-1 consumed
        if (j + 1 < nblk) issue(j + 1);
        const char *sk = s_k[0] + (j & 1) * SB, *sv = s_v[0] + (j & 1) * SB;
        const int k0 = j * kWideKeys;

        // S^T[key][query]: element i of tile c is key 32c + 8 (i / 4) + 4g + i % 4
        floatx16 st[KT];
#pragma unroll
        for (int c = 0; c < KT; ++c) {
#pragma unroll
            for (int i = 0; i < 16; ++i) st[c][i] = 0.f;
#pragma unroll
            for (int s = 0; s < DS; ++s)
                st[c] = mfma32(*reinterpret_cast<const u32x4 *>(sk + ka[s] + 32 * c * RB), qf[s], st[c]);
        }
        if (k0 + kWideKeys > vis_min) {                      // wave-uniform: some key is masked
#pragma unroll
            for (int c = 0; c < KT; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + 32 * c + 8 * (i / 4) + 4 * g + i % 4 >= vis) st[c][i] = -INFINITY;
        }
        float bm = -INFINITY;
#pragma unroll
        for (int c = 0; c < KT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) bm = fmaxf(bm, st[c][i]);
        {
            const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(bm), __float_as_uint(bm), false, false);
            bm = fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1])) * sc;
        }
        const bool raise = bm > m + kLazyRescale;
        if (__builtin_expect(__ballot(raise) != 0, 0)) {
            const float alpha = raise ? __builtin_amdgcn_exp2f(m - bm) : 1.f;
            if (raise) m = bm;
            l *= alpha;
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[t][i] *= alpha;
        }
        const float mm = m == -INFINITY ? INFINITY : m;     // nothing visible yet: every weight 0
        uint32_t pk[KT][8];
#pragma unroll
        for (int c = 0; c < KT; ++c)
#pragma unroll
            for (int i = 0; i < 16; i += 2) {
                const float p0 = __builtin_amdgcn_exp2f(fmaf(st[c][i], sc, -mm));
                const float p1 = __builtin_amdgcn_exp2f(fmaf(st[c][i + 1], sc, -mm));
                l += p0 + p1;
                pk[c][i / 2] = bf16_pair(p0, p1);
            }
        // O^T[d][query] += V^T[d][keys] P^T[keys][query], sixteen keys per product: lane
        // group g holds keys 4g + 0..3 and 8 + 4g + 0..3 of them in P, and the transposing
        // reads give the same keys of V column 32t + lane % 32.
#pragma unroll
        for (int c = 0; c < KT; ++c)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const u32x4 pb{pk[c][4 * u], pk[c][4 * u + 1], pk[c][4 * u + 2], pk[c][4 * u + 3]};
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    const u32x2 lo = read_tr_tracked(sv + va[t] + (32 * c + 16 * u) * RB);
                    const u32x2 hi = read_tr_tracked(sv + va[t] + (32 * c + 16 * u + 8) * RB);
                    o[t] = mfma32(u32x4{lo[0], lo[1], hi[0], hi[1]}, pb, o[t]);
                }
            }
    }

    {
        const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
        l = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    }
    if (!qvalid) return;
    // O^T tile t, elements 4e .. 4e + 3: d = 32t + 8e + 4g + 0..3 of this lane's query
    char *orow = static_cast<char *>(a.out) + ((static_cast<int64_t>(b) * a.n_q + r) * a.Hq + hq) * D * 2;
    const float inv = live && l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t w0 = bf16_pair(o[t][4 * e] * inv, o[t][4 * e + 1] * inv);
            const uint32_t w1 = bf16_pair(o[t][4 * e + 2] * inv, o[t][4 * e + 3] * inv);
            *reinterpret_cast<u32x2 *>(orow + (32 * t + 8 * e + 4 * g) * 2) = u32x2{w0, w1};
        }
}

// One wave per query row: merges the row's pieces.  The pieces that hold a key the row
// sees are [0, ceil(vis / chunk)); lane s weighs piece s (at most 64), then D / 4 lanes
// take one piece's four output columns each, 64 / (D / 4) pieces side by side.
template <int D>
__global__ __launch_bounds__(256) void k_attention_combine(AttnArgs a) {
    constexpr int LP = D / 4;                              // lanes of one piece
    constexpr int SP = 64 / LP;                            // pieces side by side
    constexpr int U = 4;                                   // loads in flight per lane
    const int lane = threadIdx.x & 63;
    const int64_t rows_all = static_cast<int64_t>(a.B) * a.n_q * a.Hq;
    const int64_t R = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (R >= rows_all) return;                             // whole wave leaves
    const int b = quot(a.by_seq_rows, static_cast<uint32_t>(R));
    const int r = quot(a.by_hq, static_cast<uint32_t>(R)) - static_cast<uint32_t>(b) * a.n_q;
    const int lc = max(a.ctx_len[b], 0);
    const int ln = static_cast<int>(min(static_cast<int64_t>(lc) + 2 * a.K + 3, static_cast<int64_t>(a.L)));
    const int p = a.q_start[b] + r;
    const bool live = p >= 0 && p < ln;
    const int vis = !live ? 0 : p < lc ? p + 1 : ln;
    const int n = (vis + a.chunk - 1) / a.chunk;           // <= a.splits <= 64
    float2 ml = make_float2(-INFINITY, 0.f);
    if (lane < n) ml = a.part_ml[lane * rows_all + R];
    float M = ml.x;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    const float w = ml.y > 0.f ? __builtin_amdgcn_exp2f(ml.x - M) : 0.f;
    float l = w * ml.y;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) l += __shfl_xor(l, off);
    const int c = lane % LP, sp = lane / LP;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < n; s0 += SP * U) {
        floatx4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = min(s0 + u * SP + sp, n - 1);    // unconditional: clamped
            v[u] = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(a.part_o + (s * rows_all + R) * D) + c);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u * SP + sp;
            const float ws = __shfl(w, s & 63);
            const bool in = s < n;                         // a piece counted twice by the clamp adds nothing
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = in ? fmaf(ws, v[u][k], acc[k]) : acc[k];
        }
    }
#pragma unroll
    for (int off = LP; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += __shfl_xor(acc[k], off);
    if (sp == 0) {
        const float inv = l > 0.f ? 1.f / l : 0.f;
        const u32x2 q{bf16_pair(acc[0] * inv, acc[1] * inv), bf16_pair(acc[2] * inv, acc[3] * inv)};
        *reinterpret_cast<u32x2 *>(static_cast<char *>(a.out) + (R * D + 4 * c) * 2) = q;
    }
}

// Waves of a workgroup of the 16-row kernel: as many as the group's rows need, at most
// kMaxWaves, spread evenly; at least four, the loaders among them.
int64_t attn_waves(int64_t rows) {
    const int64_t per_max = 16 * kMaxWaves;
    const int64_t nwg = (rows + per_max - 1) / per_max;
    return std::max<int64_t>(4, (((rows + nwg - 1) / nwg) + 15) / 16);
}

// Query rows of a group from which the wide kernel runs: what no longer fits one workgroup
// of the 16-row kernel (64 groups-of-8 x 132 rows x 2081 keys: 156 us there, 127 wide).
constexpr int64_t kWideMinRows = 129;
constexpr int64_t kCus = 256;         // compute units of an MI355X
constexpr int64_t kMinChunk = 128;    // keys of a piece, at least

}  // namespace

// How the keys of a call are cut: the cheapest count by a cost in microseconds whose terms
// were measured on MI355X with 68 query rows per group.  A workgroup alone on its CU takes
// t1 per key (D = 128: 256 groups x 2065 keys 47.7 us), one that shares it t2 (512 groups
// 76 us), the merge's launch 3.5 us, and each piece's sums are written and read back at
// about 3 TB/s.  The cost agrees with the measured times of 16 to 256 groups, cut 1 to 32
// times, within 3 us: 16 groups x 16401 keys 330 us uncut, 32.0 in 256 workgroups, 34.0 in
// 512; 64 x 4017 31.5 in 256, 36.1 in 512; 96 x 2517 36.9 in 192, 32.5 in 480; 160 x 4113
// 87 uncut, 79 in 320, 65 in 480; 224 x 2017 46 uncut, 53 in 448.  Short contexts are not cut:
// a call of two launches takes 13.5 us at the least (8 groups, D = 128: 417 keys 13.0 uncut, 537
// keys 15.1 uncut and 13.5 cut; D = 64: 537 keys 11.9 uncut, 717 15.1).  More groups than CUs are
// not cut: two of them already share a CU.
// From kWideMinRows rows on the uncut call runs the wide kernel, whose time with at most one
// workgroup per CU is a line in L (212 to 1048 rows, within 0.6 us: D = 128 16.6 us at 653 keys,
// 39.3 at 2053, 104.7 at 6083; D = 64 11.7, 27.7 and 73.0), and a cut must win by what its cost
// falls short of there.  64 calls of 129 rows or more, uncut and cut: one input of 2017
// positions, 16/8 heads, D = 64 27.0 and 46.2 us, 8/8 heads, D = 128 38.4 and 38.2, 1217 positions 25.3
// and 22.9; 4 x 1083 keys, 332 rows, D = 64 16.3 and 21.0; 2 x 6083 keys 73.6 and 28.2; the rule takes
// the slower one twice, by 0.4 and 0.8 us.
AttnPlan attn_plan(int32_t B, int32_t n_q, int32_t L, int32_t Hq, int32_t Hkv, int32_t D) {
    AttnPlan p{1, 0, 0};
    const int64_t rows = static_cast<int64_t>(n_q) * (Hq / Hkv);
    if (B <= 0 || rows <= 0) return p;
    const int64_t waves = attn_waves(rows);
    const int64_t wgs = static_cast<int64_t>(B) * Hkv * ((rows + 16 * waves - 1) / (16 * waves));
    if (wgs > kCus) return p;
    const double t1 = D == 128 ? 0.023 : 0.0185, t2 = D == 128 ? 0.037 : 0.022;
    const double piece_us = static_cast<double>(std::min<int64_t>(rows, 16 * waves)) * D * 8 / 3e6;
    const bool wide = rows >= kWideMinRows;
    double best = !wide ? L * t1 : D == 128 ? 5.8 + 0.01625 * L - 1.0 : 4.6 + 0.01125 * L - 2.7;
    if (best < (wide ? 13.7 : 10.5)) return p;
    for (int64_t s = 2; s <= 64 && wgs * s <= 2 * kCus; ++s) {
        const int64_t chunk = ((L + s - 1) / s + kKeyBlock - 1) / kKeyBlock * kKeyBlock;
        if (chunk < kMinChunk) break;
        const int64_t n = (L + chunk - 1) / chunk;
        const double cost = chunk * (wgs * n <= kCus ? t1 : t2) + 3.5 + piece_us * static_cast<double>(wgs * n);
        if (n < 2 || cost >= best) continue;
        best = cost;
        p.splits = static_cast<int32_t>(n);
        p.chunk = static_cast<int32_t>(chunk);
        p.rows = static_cast<int64_t>(B) * n_q * Hq;
    }
    return p;
}

hipError_t launch_hybrid_mask(const MaskArgs &a, hipStream_t s) {
    const int64_t rows = static_cast<int64_t>(a.B) * a.L;
    if (rows == 0) return hipSuccess;
    hipLaunchKernelGGL(k_hybrid_mask, dim3(static_cast<unsigned>(rows)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_hybrid_attention(AttnArgs a, hipStream_t s) {
    const int64_t rows = static_cast<int64_t>(a.n_q) * (a.Hq / a.Hkv);
    const int64_t waves = attn_waves(rows);
    const int64_t wgs = static_cast<int64_t>(a.B) * a.Hkv * ((rows + 16 * waves - 1) / (16 * waves));
    if (wgs == 0) return hipSuccess;
    const dim3 block(static_cast<unsigned>(64 * waves));
    a.by_grp = fast_div(a.Hq / a.Hkv);
    a.by_wgs = fast_div(static_cast<uint32_t>((rows + 16 * waves - 1) / (16 * waves)));
    a.by_hkv = fast_div(a.Hkv);
    a.by_splits = fast_div(a.splits);
    a.by_seq_rows = fast_div(static_cast<uint32_t>(a.n_q) * static_cast<uint32_t>(a.Hq));
    a.by_hq = fast_div(a.Hq);
    if (a.splits > 1) {
        const dim3 grid(static_cast<unsigned>(wgs * a.splits));
        const dim3 cgrid(static_cast<unsigned>((static_cast<int64_t>(a.B) * a.n_q * a.Hq + 3) / 4));
        if (a.D == 128) {
            hipLaunchKernelGGL((k_hybrid_attention<128, true>), grid, block, 0, s, a);
            hipLaunchKernelGGL(k_attention_combine<128>, cgrid, dim3(256), 0, s, a);
        } else {
            hipLaunchKernelGGL((k_hybrid_attention<64, true>), grid, block, 0, s, a);
            hipLaunchKernelGGL(k_attention_combine<64>, cgrid, dim3(256), 0, s, a);
        }
        return hipGetLastError();
    }
    if (rows >= kWideMinRows) {
        const int64_t groups = static_cast<int64_t>(a.B) * a.Hkv;
        const int64_t xcds = groups % kXcds == 0 ? kXcds : 1;
        const int64_t tiles = (rows + kWideRows - 1) / kWideRows;
        // 4 sequences x 2065 positions, 32/8 heads: 136 us tile by tile, 109 us group by
        // group; 16 x 317, 8/8 heads (384 workgroups, two to a CU): 13.7 against 15.4 us
        const bool by_tile = groups * tiles <= 2 * kCus;
        a.by_wgs = fast_div(static_cast<uint32_t>(by_tile ? groups / xcds : tiles));
        a.chunk = by_tile;
        a.splits = static_cast<int32_t>(xcds);
        const dim3 wgrid(static_cast<unsigned>(groups * tiles));
        if (a.D == 128) hipLaunchKernelGGL(k_hybrid_attention_wide<128>, wgrid, dim3(64 * kWideWaves), 0, s, a);
        else hipLaunchKernelGGL(k_hybrid_attention_wide<64>, wgrid, dim3(64 * kWideWaves), 0, s, a);
        return hipGetLastError();
    }
    const dim3 grid(static_cast<unsigned>(wgs));
    if (a.D == 128) hipLaunchKernelGGL((k_hybrid_attention<128, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_hybrid_attention<64, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace cospec
