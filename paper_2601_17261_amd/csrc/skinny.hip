// Tall-skinny products of Alg. 1 on bf16 activations (HBM-bound sweeps of X):
//   xq  : T = X Q          (N x r), contraction over d_in   -> also used for the projection P = X B
//   xtt : S = X^T T        (d_in x r), contraction over tokens (T = Omega or T = X Q)
// X is bf16; the small fp32 factor (Q, B, T, Omega) enters the matrix cores as three bf16 planes
// hi + mid + lo, whose sum is the fp32 value, so the products carry fp32-level accuracy while the
// kernels stay bound by the single read of X.  v_mfma_f32_16x16x32_bf16 throughout.
#include <algorithm>
#include <type_traits>

#include "ext_prep.h"

namespace agzo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

union Frag {
    uint4 u;
    bf16x8 v;
};

// ---------------------------------------------------------------------------
// xq: workgroup = 64 tokens, wave = 16 of them over the whole of d_in, so no cross-wave reduction.
// MFMA roles: A = X tile (rows = tokens, K = d_in), B = Q planes (K = d_in, cols = k); the three planes
// accumulate into the same registers.  X and the plane rows travel global -> LDS directly in 64-wide
// slices (one 128-byte line per row and slice, XOR-swizzled chunks) through a ring of XQ_STAGES slots,
// so that enough bytes are in flight per CU to cover the memory latency with four waves.
// ---------------------------------------------------------------------------
constexpr int kXShare = kProductsOfOneX;
// Workgroups from which on a launch of products that share an X takes them in groups.  Fewer leave compute units idle that the products by
// themselves, in smaller pieces, would use.  A step, us, without and with groups: 0.6B-sized layers on 512 tokens (56 and 112 workgroups) 226 and 254,
// on 1000 (112 and 224) 274 and 278, on 1400 326 and 312, on 2048 (194 and 448) 392 and 376; 4B-sized on 200 (74 and 136) 384 and 393, on 400 503
// and 489, on 512 (148 and 272) 535 and 521; 8B-sized on 300 (144 and 200) 711 and 683, on 16384 14749 and 14350.  2.3 layers of a
// decoder, 2048 and 6144 wide, on 8192: 116 and 94 a launch of X^T T, 112 and 109 of X Q
constexpr uint64_t XTT_GROUP_MIN = 128, XQ_GROUP_MIN = 192;

constexpr int XQ_TOK = 64;
constexpr int XQ_BK = 64;

__device__ __forceinline__ int xq_lds_off(int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); }

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// T[t][k] as the X side of the extension operands: [hi | hi | lo | 0], segments of rp columns, the last one up to the width
__device__ __forceinline__ void store_ext(bf16_t* Xext, int64_t t, int k, int rp, float v) {
    const int ld = (3 * rp + 63) / 64 * 64;
    bf16_t* dst = Xext + t * ld + k;
    const bf16_t hi = f32_to_bf16(v), lo = f32_to_bf16(v - bf16_to_f32(hi));
    dst[0] = hi; dst[rp] = hi; dst[2 * rp] = lo;
    if (3 * rp < ld) dst[3 * rp] = 0;          // (ld - 3 rp is 0 or rp)
}

// the results of tokens t .. t + 3 (t and m_pad multiples of 4), column k
__device__ __forceinline__ void xq_emit(floatx4 v, int64_t M, int r, int rp, float* __restrict__ T, bf16_t* __restrict__ TpackT, int64_t m_pad,
                                        bf16_t* __restrict__ Xext, int64_t t, int k) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (!(t + e < M && k < r)) v[e] = 0.f;
        if (t + e < M && k < r && T != nullptr) T[(t + e) * r + k] = v[e];
        if (t + e < M && Xext != nullptr) store_ext(Xext, t + e, k, rp, v[e]);
    }
    if (TpackT == nullptr || t >= m_pad) return;
    uint32_t w[3][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        bf16_t h[2], m[2], l[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) split3_bf16(v[2 * u + i], h[i], m[i], l[i]);
        w[0][u] = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
        w[1][u] = (uint32_t)m[0] | ((uint32_t)m[1] << 16);
        w[2][u] = (uint32_t)l[0] | ((uint32_t)l[1] << 16);
    }
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2*>(TpackT + ((int64_t)pl * rp + k) * m_pad + t) = make_uint2(w[pl][0], w[pl][1]);
}
// what a wave's accumulators become.  D layout: row (token) = 4*(lane/16) + e, col (k) = lane%16.  part: partial sums, column by
// column where planes are to be written, [split][RP][m_pad], token by token otherwise, [split][m_pad][RP]
template <int NB, int MB>
__device__ __forceinline__ void xq_store(const floatx4 (&acc)[MB][NB], int64_t M, int r, float* __restrict__ T, bf16_t* __restrict__ TpackT, int64_t m_pad,
                                         float* __restrict__ part, bf16_t* __restrict__ Xext, int64_t t0, int split, int wave, int lm, int lg) {
    constexpr int RP = NB * 16;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int64_t t = t0 + (wave * MB + mb) * 16 + lg * 4;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int k = nb * 16 + lm;
            if (part == nullptr) xq_emit(acc[mb][nb], M, r, RP, T, TpackT, m_pad, Xext, t, k);
            else if (t >= m_pad) continue;
            else if (TpackT != nullptr) *reinterpret_cast<floatx4*>(part + ((int64_t)split * RP + k) * m_pad + t) = acc[mb][nb];
            else
#pragma unroll
                for (int e = 0; e < 4; ++e) part[((int64_t)split * m_pad + t + e) * RP + k] = acc[mb][nb][e];
        }
    }
}

// bx: token block, by / ny: this workgroup's share of d_in (ny = 1: all of it)
// ring depth: DEEP = 1, one workgroup per CU with as many slices in flight as LDS holds; 0, a shallower ring that
// lets two workgroups share a CU, for launches with at least two workgroups per CU (several layers at once): while one
// waits at its barrier or on its fragment reads the other multiplies; 2, what a workgroup of the forwards leaves of the LDS
template <int NB, int DEEP>
struct XqRing { static constexpr int STAGES = DEEP == 1 ? (NB == 1 ? 8 : 6) : NB == 2 ? 3 : DEEP == 2 ? 4 : 5; };

// a slot holds the rows of a slice and, where four waves do not share their groups evenly, groups that nobody reads: every wave
// then issues the same number of loads and waits by constants (a wait chosen among a dozen cases and a branch around each load
// cost more than the slice's matrix work)
constexpr int xq_slot_bytes(int nb) { return (XQ_TOK / 8 + 6 * nb + 3) / 4 * 4096; }

template <int NB, int DEEP>
__device__ __forceinline__ void xq_bf16_body(const bf16_t* __restrict__ X, int64_t ldx, int64_t M, int64_t K,
                                             const bf16_t* __restrict__ Qpack, int r, float* __restrict__ T,
                                             bf16_t* __restrict__ TpackT, int64_t m_pad, float* __restrict__ part,
                                             bf16_t* __restrict__ Xext, uint32_t bx, uint32_t by, uint32_t ny) {
    constexpr int RP = NB * 16;
    constexpr int QROWS = 3 * RP;                          // plane rows: (plane, k)
    constexpr int NGROUP = XQ_TOK / 8 + QROWS / 8;         // 8-row groups per slice: X first, then the planes
    constexpr int SLOT = xq_slot_bytes(NB);                // bytes per ring slot
    constexpr int STAGES = XqRing<NB, DEEP>::STAGES;
    extern __shared__ __align__(16) char xq_smem[];
    typedef __attribute__((address_space(3))) void* lptr_t;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lg = lane >> 4;
    const int64_t t0 = (int64_t)bx * XQ_TOK;

    floatx4 acc[1][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[0][nb] = floatx4{0.f, 0.f, 0.f, 0.f};

    // this wave's row groups g = wave, wave + 4, ...: per-lane source pointers (row of the group, swizzled chunk)
    constexpr int MAXG = (NGROUP + 3) / 4;
    const bf16_t* src[MAXG];
#pragma unroll
    for (int i = 0; i < MAXG; ++i) {
        const int g = min(wave + 4 * i, NGROUP - 1);
        const int row = 8 * g + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        if (row < XQ_TOK) src[i] = X + min(t0 + row, M - 1) * ldx + c * 8;
        else src[i] = Qpack + (int64_t)(row - XQ_TOK) * K + c * 8;
    }
    // few tokens: gridDim.y workgroups share a token block, each taking a contiguous run of d_in slices, and leave
    // partial sums in `part` for xq_finish_many_kernel (a single workgroup per block would walk d_in alone, bound by latency)
    const int nsplit = (int)ny, split = (int)by;
    const int nfull_all = (int)(K / XQ_BK);
    const int kbeg = (int)((int64_t)nfull_all * split / nsplit);
    const int nfull = (int)((int64_t)nfull_all * (split + 1) / nsplit) - kbeg;      // this workgroup's slices
    const bool tail = (K % XQ_BK) != 0 && split == nsplit - 1;
#pragma unroll
    for (int i = 0; i < MAXG; ++i) src[i] += (int64_t)kbeg * XQ_BK;
    // the next slice not yet requested, into `slot`
    auto issue = [&](int slot) __attribute__((always_inline)) {
        char* base = xq_smem + slot * SLOT + wave * 1024;
#pragma unroll
        for (int i = 0; i < MAXG; ++i) {
            __builtin_amdgcn_global_load_lds((gptr_t)src[i], (lptr_t)(base + i * 4096), 16, 0, 0);
            src[i] += XQ_BK;
        }
    };
    // Fragment reads go through inline assembly: for a plain LDS load the compiler, which cannot tell the ring's slots
    // apart, first waits for every direct load in flight (vmcnt(0)) and so collapses the ring to one slice.  The reads of a
    // slice, both of its 32-wide sub-steps, and the wait for them are one block: with one workgroup per compute unit a slice is
    // a chain of LDS latency and dependent matrix instructions, and one latency is less than two.
    // Row 16 m + lm of an operand lies 2048 m bytes behind row lm, in the same chunk order.
    auto multiply = [&](int slot) __attribute__((always_inline)) {
        const char* xs = xq_smem + slot * SLOT;
        const char* qs = xs + XQ_TOK * 128;
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 a[2], b[2][NB][3];
        const uint32_t xaddr0 = (uint32_t)(uintptr_t)(lptr_t)(xs + xq_lds_off(wave * 16 + lm, lg)), xaddr1 = (uint32_t)(uintptr_t)(lptr_t)(xs + xq_lds_off(wave * 16 + lm, 4 + lg));
        const uint32_t qaddr0 = (uint32_t)(uintptr_t)(lptr_t)(qs + xq_lds_off(lm, lg)), qaddr1 = (uint32_t)(uintptr_t)(lptr_t)(qs + xq_lds_off(lm, 4 + lg));
        static_assert(NB <= 2, "wider ones read X directly");
        if constexpr (NB == 1)
            asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %10 offset:2048\n\t"
                         "ds_read_b128 %4, %10 offset:4096\n\tds_read_b128 %1, %9\n\tds_read_b128 %5, %11\n\t"
                         "ds_read_b128 %6, %11 offset:2048\n\tds_read_b128 %7, %11 offset:4096\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0][0][0]), "=&v"(b[0][0][1]), "=&v"(b[0][0][2]),
                           "=&v"(b[1][0][0]), "=&v"(b[1][0][1]), "=&v"(b[1][0][2])
                         : "v"(xaddr0), "v"(xaddr1), "v"(qaddr0), "v"(qaddr1) : "memory");
        else
            asm volatile("ds_read_b128 %0, %14\n\tds_read_b128 %2, %16\n\tds_read_b128 %3, %16 offset:2048\n\t"
                         "ds_read_b128 %4, %16 offset:4096\n\tds_read_b128 %5, %16 offset:6144\n\t"
                         "ds_read_b128 %6, %16 offset:8192\n\tds_read_b128 %7, %16 offset:10240\n\tds_read_b128 %1, %15\n\t"
                         "ds_read_b128 %8, %17\n\tds_read_b128 %9, %17 offset:2048\n\tds_read_b128 %10, %17 offset:4096\n\t"
                         "ds_read_b128 %11, %17 offset:6144\n\tds_read_b128 %12, %17 offset:8192\n\t"
                         "ds_read_b128 %13, %17 offset:10240\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0][0][0]), "=&v"(b[0][1][0]), "=&v"(b[0][0][1]),
                           "=&v"(b[0][1][1]), "=&v"(b[0][0][2]), "=&v"(b[0][1][2]), "=&v"(b[1][0][0]), "=&v"(b[1][1][0]),
                           "=&v"(b[1][0][1]), "=&v"(b[1][1][1]), "=&v"(b[1][0][2]), "=&v"(b[1][1][2])
                         : "v"(xaddr0), "v"(xaddr1), "v"(qaddr0), "v"(qaddr1) : "memory");
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[sub]), __builtin_bit_cast(bf16x8, b[sub][nb][pl]),
                                                                         acc[0][nb], 0, 0, 0);
    };
    // ring: slices kt .. kt + STAGES - 2 in flight while slice kt is multiplied
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < nfull) issue(s);
    int slot = 0;
    // the slice in `slot`, with YOUNGER slices in flight behind it
    auto step = [&](auto YOUNGER, bool more) __attribute__((always_inline)) {
        wait_vmcnt<decltype(YOUNGER)::value * MAXG>();     // this wave's loads of the slice have landed
        // everybody's have; the slot of the slice before is free.  A bare barrier: __syncthreads()
        // would first wait for every load in flight and collapse the ring to one slice.
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue(slot == 0 ? STAGES - 1 : slot - 1);
        multiply(slot);
        slot = (slot + 1 == STAGES) ? 0 : slot + 1;
    };
    const int rest = min(nfull, STAGES - 1);
    for (int kt = 0; kt < nfull - rest; ++kt) step(std::integral_constant<int, STAGES - 2>{}, true);
    auto drain = [&](auto self, auto YOUNGER) __attribute__((always_inline)) -> void {
        constexpr int y = decltype(YOUNGER)::value;
        if (y < rest) step(YOUNGER, false);
        if constexpr (y > 0) self(self, std::integral_constant<int, y - 1>{});
    };
    drain(drain, std::integral_constant<int, STAGES - 2>{});
    if (tail) {
        // ragged end of d_in: the threads copy it themselves, zero past d_in
        __syncthreads();
        char* base = xq_smem;                              // slot 0 (all loads have landed and were consumed)
        for (int e = tid; e < (XQ_TOK + QROWS) * 8; e += 256) {
            const int row = e >> 3, c = e & 7;
            const int64_t kcol = (int64_t)nfull_all * XQ_BK + c * 8;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (kcol < K) {
                const bf16_t* p = (row < XQ_TOK) ? X + min(t0 + row, M - 1) * ldx + kcol
                                                 : Qpack + (int64_t)(row - XQ_TOK) * K + kcol;
                v = *reinterpret_cast<const uint4*>(p);
            }
            *reinterpret_cast<uint4*>(base + xq_lds_off(row, c)) = v;
        }
        __syncthreads();
        multiply(0);
    }
    // (Copies that the compiler cannot see through: with the accumulators themselves in the epilogue it swapped the two of 32 columns every
    // slice, twelve moves and a wait beside twelve matrix instructions; one layer 4096 wide, r = 32, on 8192 tokens: 63.6 us a perturbed
    // forward and 61)
    floatx4 res[1][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float x = acc[0][nb][e];
            asm volatile("" : "+v"(x));
            res[0][nb][e] = x;
        }
    xq_store<NB, 1>(res, M, r, T, TpackT, m_pad, part, Xext, t0, split, wave, lm, lg);
}

// 48 and 64 columns.  The rows of X, which one wave alone reads, go to its registers, and only the planes through LDS: three
// slices of them leave room for two workgroups on a compute unit.  A slice's 32-wide sub-steps take 16-byte chunks 2 lg and
// 2 lg + 1 of a row, so that a row's line is asked for at once.  MB = 2, a wave with 32 tokens, reads the planes half as often: at 64
// columns every wave reads 24 KB of them from LDS a slice against 2 KB of its own 16 tokens (4096 tokens of seven 4B-sized layers, r =
// 64: 86 us through the ring above, 74 and 62 here with MB = 1 and 2)
constexpr int XQD_STAGES = 3;
constexpr int xqd_loads(int nb) { return (6 * nb + 3) / 4; }
template <int NB, int MB>
__device__ __forceinline__ void xq_direct_body(const bf16_t* __restrict__ X, int64_t ldx, int64_t M, int64_t K,
                                               const bf16_t* __restrict__ Qpack, int r, float* __restrict__ T,
                                               bf16_t* __restrict__ TpackT, int64_t m_pad, float* __restrict__ part,
                                               bf16_t* __restrict__ Xext, uint32_t bx, uint32_t by, uint32_t ny) {
    constexpr int RP = NB * 16, TOK = MB * XQ_TOK;
    constexpr int QROWS = 3 * RP, LOADS = xqd_loads(NB);                // plane rows; a wave's direct loads of a slice
    constexpr int STAGES = XQD_STAGES, SLOT = LOADS * 4096;
    extern __shared__ __align__(16) char xq_smem[];
    typedef __attribute__((address_space(3))) void* lptr_t;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lg = lane >> 4;
    const int64_t t0 = (int64_t)bx * TOK;

    floatx4 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int nsplit = (int)ny, split = (int)by;
    const int nfull_all = (int)(K / XQ_BK);
    const int kbeg = (int)((int64_t)nfull_all * split / nsplit);
    const int nfull = (int)((int64_t)nfull_all * (split + 1) / nsplit) - kbeg;      // this workgroup's slices
    const bool tail = (K % XQ_BK) != 0 && split == nsplit - 1;
    // plane rows: groups of eight, wave w takes w, w + 4, ... (past the last: the last once more, into rows nobody reads)
    const bf16_t* src[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int row = 8 * (wave + 4 * i) + (lane >> 3);
        src[i] = Qpack + (int64_t)min(row, QROWS - 8 + (lane >> 3)) * K + ((lane & 7) ^ ((row >> 1) & 7)) * 8 + (int64_t)kbeg * XQ_BK;
    }
    const bf16_t* xsrc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) xsrc[mb] = X + min(t0 + (wave * MB + mb) * 16 + lm, M - 1) * ldx + lg * 16 + (int64_t)kbeg * XQ_BK;
    u32x4 x[STAGES][MB][2];
    auto issue = [&](auto SET) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value;
        char* base = xq_smem + set * SLOT + wave * 1024;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            __builtin_amdgcn_global_load_lds((gptr_t)src[i], (lptr_t)(base + i * 4096), 16, 0, 0);
            src[i] += XQ_BK;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) x[set][mb][sub] = *reinterpret_cast<const u32x4*>(xsrc[mb] + sub * 8);
            xsrc[mb] += XQ_BK;
        }
    };
    auto multiply = [&](int slot, u32x4 (&xa)[MB][2]) __attribute__((always_inline)) {
        const char* qs = xq_smem + slot * SLOT;
        u32x4 b[2][NB][3];
        const uint32_t qaddr0 = (uint32_t)(uintptr_t)(lptr_t)(qs + xq_lds_off(lm, 2 * lg)), qaddr1 = (uint32_t)(uintptr_t)(lptr_t)(qs + xq_lds_off(lm, 2 * lg + 1));
        static_assert(NB == 3 || NB == 4, "column blocks");
        if constexpr (NB == 3)
            asm volatile("ds_read_b128 %0, %18\n\tds_read_b128 %1, %18 offset:2048\n\tds_read_b128 %2, %18 offset:4096\n\t"
                                     "ds_read_b128 %3, %18 offset:6144\n\tds_read_b128 %4, %18 offset:8192\n\tds_read_b128 %5, %18 offset:10240\n\t"
                                     "ds_read_b128 %6, %18 offset:12288\n\tds_read_b128 %7, %18 offset:14336\n\tds_read_b128 %8, %18 offset:16384\n\t"
                                     "ds_read_b128 %9, %19\n\tds_read_b128 %10, %19 offset:2048\n\tds_read_b128 %11, %19 offset:4096\n\t"
                                     "ds_read_b128 %12, %19 offset:6144\n\tds_read_b128 %13, %19 offset:8192\n\tds_read_b128 %14, %19 offset:10240\n\t"
                                     "ds_read_b128 %15, %19 offset:12288\n\tds_read_b128 %16, %19 offset:14336\n\tds_read_b128 %17, %19 offset:16384\n\t"
                                     "s_waitcnt lgkmcnt(0)"
                                     : "=&v"(b[0][0][0]), "=&v"(b[0][1][0]), "=&v"(b[0][2][0]), "=&v"(b[0][0][1]), "=&v"(b[0][1][1]),
                                       "=&v"(b[0][2][1]), "=&v"(b[0][0][2]), "=&v"(b[0][1][2]), "=&v"(b[0][2][2]), "=&v"(b[1][0][0]),
                                       "=&v"(b[1][1][0]), "=&v"(b[1][2][0]), "=&v"(b[1][0][1]), "=&v"(b[1][1][1]), "=&v"(b[1][2][1]),
                                       "=&v"(b[1][0][2]), "=&v"(b[1][1][2]), "=&v"(b[1][2][2])
                                     : "v"(qaddr0), "v"(qaddr1) : "memory");
        else
            asm volatile("ds_read_b128 %0, %24\n\tds_read_b128 %1, %24 offset:2048\n\tds_read_b128 %2, %24 offset:4096\n\t"
                                     "ds_read_b128 %3, %24 offset:6144\n\tds_read_b128 %4, %24 offset:8192\n\tds_read_b128 %5, %24 offset:10240\n\t"
                                     "ds_read_b128 %6, %24 offset:12288\n\tds_read_b128 %7, %24 offset:14336\n\tds_read_b128 %8, %24 offset:16384\n\t"
                                     "ds_read_b128 %9, %24 offset:18432\n\tds_read_b128 %10, %24 offset:20480\n\tds_read_b128 %11, %24 offset:22528\n\t"
                                     "ds_read_b128 %12, %25\n\tds_read_b128 %13, %25 offset:2048\n\tds_read_b128 %14, %25 offset:4096\n\t"
                                     "ds_read_b128 %15, %25 offset:6144\n\tds_read_b128 %16, %25 offset:8192\n\tds_read_b128 %17, %25 offset:10240\n\t"
                                     "ds_read_b128 %18, %25 offset:12288\n\tds_read_b128 %19, %25 offset:14336\n\tds_read_b128 %20, %25 offset:16384\n\t"
                                     "ds_read_b128 %21, %25 offset:18432\n\tds_read_b128 %22, %25 offset:20480\n\tds_read_b128 %23, %25 offset:22528\n\t"
                                     "s_waitcnt lgkmcnt(0)"
                                     : "=&v"(b[0][0][0]), "=&v"(b[0][1][0]), "=&v"(b[0][2][0]), "=&v"(b[0][3][0]), "=&v"(b[0][0][1]),
                                       "=&v"(b[0][1][1]), "=&v"(b[0][2][1]), "=&v"(b[0][3][1]), "=&v"(b[0][0][2]), "=&v"(b[0][1][2]),
                                       "=&v"(b[0][2][2]), "=&v"(b[0][3][2]), "=&v"(b[1][0][0]), "=&v"(b[1][1][0]), "=&v"(b[1][2][0]),
                                       "=&v"(b[1][3][0]), "=&v"(b[1][0][1]), "=&v"(b[1][1][1]), "=&v"(b[1][2][1]), "=&v"(b[1][3][1]),
                                       "=&v"(b[1][0][2]), "=&v"(b[1][1][2]), "=&v"(b[1][2][2]), "=&v"(b[1][3][2])
                                     : "v"(qaddr0), "v"(qaddr1) : "memory");
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[mb][sub]), __builtin_bit_cast(bf16x8, b[sub][nb][pl]),
                                                                              acc[mb][nb], 0, 0, 0);
    };
    // slices kt .. kt + 2: one being multiplied, two in flight
    std::integral_constant<int, 0> c0; std::integral_constant<int, 1> c1; std::integral_constant<int, 2> c2;
    auto step = [&](auto SET, auto YOUNGER, bool more) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value;
        wait_vmcnt<decltype(YOUNGER)::value * (LOADS + 2 * MB)>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue(std::integral_constant<int, (set + 2) % 3>{});
        __builtin_amdgcn_sched_barrier(0);
        multiply(set, x[set]);
    };
    if (nfull >= 2) {
        issue(c0);
        __builtin_amdgcn_sched_barrier(0);
        issue(c1);
        __builtin_amdgcn_sched_barrier(0);
        int left = nfull;
        for (; left >= 5; left -= 3) {
            step(c0, c1, true);
            step(c1, c1, true);
            step(c2, c1, true);
        }
        if (left == 4) { step(c0, c1, true); step(c1, c1, true); step(c2, c1, false); step(c0, c0, false); }
        else if (left == 3) { step(c0, c1, true); step(c1, c1, false); step(c2, c0, false); }
        else { step(c0, c1, false); step(c1, c0, false); }
    } else if (nfull == 1) {
        issue(c0);
        step(c0, c0, false);
    }
    if (tail) {
        // ragged end of d_in: the threads copy it themselves, zero past d_in
        __syncthreads();
        const int64_t k0 = (int64_t)nfull_all * XQ_BK;
        for (int e = tid; e < QROWS * 8; e += 256) {
            const int row = e >> 3, c = e & 7;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (k0 + c * 8 < K) v = *reinterpret_cast<const uint4*>(Qpack + (int64_t)row * K + k0 + c * 8);
            *reinterpret_cast<uint4*>(xq_smem + xq_lds_off(row, c)) = v;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
                const int64_t k = k0 + lg * 16 + sub * 8;
                u32x4 v = {0, 0, 0, 0};
                if (k < K) v = *reinterpret_cast<const u32x4*>(X + min(t0 + (wave * MB + mb) * 16 + lm, M - 1) * ldx + k);
                x[0][mb][sub] = v;
            }
        __syncthreads();
        multiply(0, x[0]);
    }
    xq_store<NB, MB>(acc, M, r, T, TpackT, m_pad, part, Xext, t0, split, wave, lm, lg);
}

// what a launch needs per product (the layers of a model)
struct XqDev {
    const bf16_t* X; int64_t ldx, M, K;
    const bf16_t* Qpack; int r;
    float* T; bf16_t* TpackT; int64_t m_pad; float* part;   // part: NULL unless ns > 1
    int ns;
    bf16_t* Xext;
};
template <int NB, int DEEP, int CAP>
__global__ __launch_bounds__(256) void xq_bf16_many_kernel(const KBatch<XqDev, CAP> tb) {
    uint32_t bx, by;
    const XqDev& a = tb.a[kbatch_find(tb, bx, by)];
    xq_bf16_body<NB, DEEP>(a.X, a.ldx, a.M, a.K, a.Qpack, a.r, a.T, a.TpackT, a.m_pad, a.part, a.Xext, bx, by, (uint32_t)a.ns);
}

template <int NB, int MB, int CAP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void xq_direct_many_kernel(const KBatch<XqDev, CAP> tb) {
    uint32_t bx, by;
    const XqDev& a = tb.a[kbatch_find(tb, bx, by)];
    xq_direct_body<NB, MB>(a.X, a.ldx, a.M, a.K, a.Qpack, a.r, a.T, a.TpackT, a.m_pad, a.part, a.Xext, bx, by, (uint32_t)a.ns);
}

// Products of several layers that read the same activations, up to four with up to 16 columns each: X is read once for all of them.  As
// xq_direct_body() with the planes of NB products side by side, in the slices' order of xq_bf16_body() (16-byte chunks lg and 4 + lg of a row's
// line): sums and bits are those of a product by itself, in whose form (xq_bf16_body()) the same launch makes those that share theirs with none.
// Bound by what a compute unit takes in, planes and X, and by the 16 rows that a load of X touches
struct XqGroupDev {
    const bf16_t* X; int64_t ldx, M, K, m_pad;
    int ns, nb;
    const bf16_t* Qpack[kXShare];
    float* T[kXShare]; bf16_t* TpackT[kXShare]; float* part[kXShare]; bf16_t* Xext[kXShare];
    int r[kXShare];
};
template <int NB, int MB>
__device__ __forceinline__ void xq_group_body(const XqGroupDev& a, uint32_t bx, uint32_t by) {
    constexpr int TOK = MB * XQ_TOK, QROWS = 48 * NB, LOADS = xqd_loads(NB);      // plane rows; a wave's direct loads of a slice
    constexpr int STAGES = XQD_STAGES, SLOT = LOADS * 4096;
    extern __shared__ __align__(16) char xq_smem[];
    typedef __attribute__((address_space(3))) void* lptr_t;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lg = lane >> 4;
    const int64_t t0 = (int64_t)bx * TOK, M = a.M, K = a.K;

    floatx4 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int nsplit = a.ns, split = (int)by;
    const int nfull_all = (int)(K / XQ_BK);
    const int kbeg = (int)((int64_t)nfull_all * split / nsplit);
    const int nfull = (int)((int64_t)nfull_all * (split + 1) / nsplit) - kbeg;      // this workgroup's slices
    const bool tail = (K % XQ_BK) != 0 && split == nsplit - 1;
    // plane rows, 16 of plane pl of product nb at 16 (pl NB + nb), in groups of eight: wave w takes w, w + 4, ... (past the last: the last once
    // more, into rows nobody reads)
    auto plane_row = [&](int row) __attribute__((always_inline)) { return a.Qpack[(row >> 4) % NB] + (int64_t)((row >> 4) / NB * 16 + (row & 15)) * K; };
    const bf16_t* src[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int group = min(wave + 4 * i, QROWS / 8 - 1), row = 8 * (wave + 4 * i) + (lane >> 3);
        src[i] = a.Qpack[(group >> 1) % NB] + (int64_t)((group >> 1) / NB * 16 + 8 * (group & 1) + (lane >> 3)) * K + ((lane & 7) ^ ((row >> 1) & 7)) * 8 + (int64_t)kbeg * XQ_BK;
    }
    const bf16_t* xsrc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) xsrc[mb] = a.X + min(t0 + (wave * MB + mb) * 16 + lm, M - 1) * a.ldx + lg * 8 + (int64_t)kbeg * XQ_BK;
    u32x4 x[STAGES][MB][2];
    auto issue = [&](auto SET) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value;
        char* base = xq_smem + set * SLOT + wave * 1024;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            __builtin_amdgcn_global_load_lds((gptr_t)src[i], (lptr_t)(base + i * 4096), 16, 0, 0);
            src[i] += XQ_BK;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) x[set][mb][sub] = *reinterpret_cast<const u32x4*>(xsrc[mb] + sub * 32);
            xsrc[mb] += XQ_BK;
        }
    };
    // (the fragments of one 32-wide sub-step at a time, reads and wait in one block)
    auto multiply = [&](int slot, u32x4 (&xa)[MB][2]) __attribute__((always_inline)) {
        const char* qs = xq_smem + slot * SLOT;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            u32x4 b[3][NB];
            const uint32_t at = (uint32_t)(uintptr_t)(lptr_t)(qs + xq_lds_off(lm, 4 * sub + lg));
            if constexpr (NB == 1)
                asm volatile("ds_read_b128 %0, %3\n\tds_read_b128 %1, %3 offset:2048\n\tds_read_b128 %2, %3 offset:4096\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(b[0][0]), "=&v"(b[1][0]), "=&v"(b[2][0]) : "v"(at) : "memory");
            else if constexpr (NB == 2)
                asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %6 offset:2048\n\tds_read_b128 %2, %6 offset:4096\n\t"
                             "ds_read_b128 %3, %6 offset:6144\n\tds_read_b128 %4, %6 offset:8192\n\tds_read_b128 %5, %6 offset:10240\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[1][0]), "=&v"(b[1][1]), "=&v"(b[2][0]), "=&v"(b[2][1]) : "v"(at) : "memory");
            else if constexpr (NB == 3)
                asm volatile("ds_read_b128 %0, %9\n\tds_read_b128 %1, %9 offset:2048\n\tds_read_b128 %2, %9 offset:4096\n\t"
                             "ds_read_b128 %3, %9 offset:6144\n\tds_read_b128 %4, %9 offset:8192\n\tds_read_b128 %5, %9 offset:10240\n\t"
                             "ds_read_b128 %6, %9 offset:12288\n\tds_read_b128 %7, %9 offset:14336\n\tds_read_b128 %8, %9 offset:16384\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[0][2]), "=&v"(b[1][0]), "=&v"(b[1][1]), "=&v"(b[1][2]),
                               "=&v"(b[2][0]), "=&v"(b[2][1]), "=&v"(b[2][2]) : "v"(at) : "memory");
            else
                asm volatile("ds_read_b128 %0, %12\n\tds_read_b128 %1, %12 offset:2048\n\tds_read_b128 %2, %12 offset:4096\n\t"
                             "ds_read_b128 %3, %12 offset:6144\n\tds_read_b128 %4, %12 offset:8192\n\tds_read_b128 %5, %12 offset:10240\n\t"
                             "ds_read_b128 %6, %12 offset:12288\n\tds_read_b128 %7, %12 offset:14336\n\tds_read_b128 %8, %12 offset:16384\n\t"
                             "ds_read_b128 %9, %12 offset:18432\n\tds_read_b128 %10, %12 offset:20480\n\tds_read_b128 %11, %12 offset:22528\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(b[0][0]), "=&v"(b[0][1]), "=&v"(b[0][2]), "=&v"(b[0][3]), "=&v"(b[1][0]), "=&v"(b[1][1]),
                               "=&v"(b[1][2]), "=&v"(b[1][3]), "=&v"(b[2][0]), "=&v"(b[2][1]), "=&v"(b[2][2]), "=&v"(b[2][3]) : "v"(at) : "memory");
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xa[mb][sub]), __builtin_bit_cast(bf16x8, b[pl][nb]),
                                                                              acc[mb][nb], 0, 0, 0);
        }
    };
    // the slices behind the one being multiplied are in flight, STAGES - 1 of them; at the end all that is left is waited for at once
    auto step = [&](auto SET, int k) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value;
        if (nfull - k > STAGES - 2) wait_vmcnt<(STAGES - 2) * (LOADS + 2 * MB)>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (nfull - k > STAGES - 1) issue(std::integral_constant<int, (set + STAGES - 1) % STAGES>{});
        __builtin_amdgcn_sched_barrier(0);
        multiply(set, x[set]);
    };
    std::integral_constant<int, 0> c0; std::integral_constant<int, 1> c1; std::integral_constant<int, 2> c2;
    static_assert(STAGES == 3, "sets");
    if (nfull > 0) issue(c0);
    __builtin_amdgcn_sched_barrier(0);
    if (nfull > 1) issue(c1);
    __builtin_amdgcn_sched_barrier(0);
    for (int k = 0; k < nfull; k += STAGES) {
        step(c0, k);
        if (k + 1 >= nfull) break;
        step(c1, k + 1);
        if (k + 2 < nfull) step(c2, k + 2);
    }
    if (tail) {
        // ragged end of d_in: the threads copy it themselves, zero past d_in
        __syncthreads();
        const int64_t k0 = (int64_t)nfull_all * XQ_BK;
        for (int e = tid; e < QROWS * 8; e += 256) {
            const int row = e >> 3, c = e & 7;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (k0 + c * 8 < K) v = *reinterpret_cast<const uint4*>(plane_row(row) + k0 + c * 8);
            *reinterpret_cast<uint4*>(xq_smem + xq_lds_off(row, c)) = v;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) {
                const int64_t k = k0 + lg * 8 + sub * 32;
                u32x4 v = {0, 0, 0, 0};
                if (k < K) v = *reinterpret_cast<const u32x4*>(a.X + min(t0 + (wave * MB + mb) * 16 + lm, M - 1) * a.ldx + k);
                x[0][mb][sub] = v;
            }
        __syncthreads();
        multiply(0, x[0]);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        floatx4 one[MB][1];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) one[mb][0] = acc[mb][nb];
        xq_store<1, MB>(one, M, a.r[nb], a.T[nb], a.TpackT[nb], a.m_pad, a.part[nb], a.Xext[nb], t0, split, wave, lm, lg);
    }
}
// HALF_CU: within what forwards on another stream leave of the LDS
template <bool HALF_CU>
constexpr int xq_group_smem(int most) { return std::max(XqRing<1, HALF_CU ? 2 : 0>::STAGES * xq_slot_bytes(1), XQD_STAGES * xqd_loads(most) * 4096); }
static_assert(xq_group_smem<false>(kXShare) <= 80 * 1024 && xq_group_smem<true>(kXShare) <= 72 * 1024, "two workgroups to a compute unit, one beside forwards");
template <int MB, bool HALF_CU>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void xq_group_kernel(const KBatch<XqGroupDev> tb) {
    uint32_t bx, by;
    const XqGroupDev& a = tb.a[kbatch_find(tb, bx, by)];
    switch (a.nb) {
        case 1: xq_bf16_body<1, HALF_CU ? 2 : 0>(a.X, a.ldx, a.M, a.K, a.Qpack[0], a.r[0], a.T[0], a.TpackT[0], a.m_pad, a.part[0], a.Xext[0], bx, by, (uint32_t)a.ns); break;
        case 2: xq_group_body<2, MB>(a, bx, by); break;
        case 3: xq_group_body<3, MB>(a, bx, by); break;
        default: xq_group_body<4, MB>(a, bx, by); break;
    }
}
static_assert(sizeof(KBatch<XqGroupDev>) <= 4096, "kernel arguments");

// sums the d_in splits of xq in fixed order and writes what the unsplit kernel's epilogue writes.  For the planes a workgroup takes
// 64 tokens of 16 columns and a thread four tokens of a column, so that the stores of a wave are whole rows (with a thread per value,
// columns side by side, every plane was written in 2-byte pieces: 28 us for 4096 tokens of seven layers at r = 64, 9 so).  T and the
// extension operands are token by token, as their partial sums are: 16 tokens of 16 columns, a thread a value, the operands then from LDS
// in 16-byte pieces.  (A thread for eight columns, 1009 tokens of a 7568-wide layer, r = 8: 4.4 us in eight workgroups and 3.1 so)
constexpr int XQF_TOK = 64, XQF_TOK_ROWS = 16;
__device__ __forceinline__ void xq_finish_body(const XqDev& a, int rp, uint32_t bx, uint32_t by) {
    const int tid = threadIdx.x, nsplit = a.ns, r = a.r;
    const int64_t m_pad = a.m_pad, M = a.M;
    // (eight splits' loads in flight; conditional on uniform values only - around a lane's condition the compiler waits for each
    // load before the next - and what lies behind the last token or column is left out below)
    if (a.TpackT != nullptr) {
        const int k = (int)by * 16 + (tid >> 4);
        const int64_t t = (int64_t)bx * XQF_TOK + 4 * (tid & 15);
        const float* src = a.part + (int64_t)k * m_pad + min(t, m_pad - 4);
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < nsplit; s0 += 8) {
            floatx4 x[8];
#pragma unroll
            for (int s = 0; s < 8; ++s)
                x[s] = s0 + s < nsplit ? *reinterpret_cast<const floatx4*>(src + (int64_t)(s0 + s) * rp * m_pad) : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 8; ++s) v += x[s];
        }
        xq_emit(v, M, r, rp, a.T, a.TpackT, m_pad, a.Xext, t, k);
        return;
    }
    __shared__ float block[XQF_TOK_ROWS][20];
    const int64_t t = (int64_t)bx * XQF_TOK_ROWS + (tid >> 4);
    const int k = (int)by * 16 + (tid & 15);
    float v = 0.f;
    const float* src = a.part + min(t, m_pad - 1) * rp + k;
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
        float x[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) x[s] = s0 + s < nsplit ? src[(int64_t)(s0 + s) * m_pad * rp] : 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) v += x[s];
    }
    if (k >= r) v = 0.f;
    if (t < M && k < r && a.T != nullptr) a.T[t * r + k] = v;
    if (a.Xext == nullptr) return;
    block[tid >> 4][tid & 15] = v;
    __syncthreads();
    const int64_t te = (int64_t)bx * XQF_TOK_ROWS + (tid >> 1);
    if (tid >= 2 * XQF_TOK_ROWS || te >= M) return;
    float c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = block[tid >> 1][8 * (tid & 1) + i];
    uint4 hi, lo;
    ext_split(c, hi, lo);
    const int ext_ld = (3 * rp + 63) / 64 * 64;
    ext_store(a.Xext + te * ext_ld, ext_ld, rp, (int)by * 16 + 8 * (tid & 1), hi, hi, lo);
}
template <int CAP>
__global__ __launch_bounds__(256) void xq_finish_many_kernel(const KBatch<XqDev, CAP> tb, int rp) {
    uint32_t bx, by;
    const XqDev& a = tb.a[kbatch_find(tb, bx, by)];
    xq_finish_body(a, rp, bx, by);
}
// with the W sides of forwards' extension operands: behind a projection both are bound by a launch's latency (4.7 + 5.6 us for 3001 tokens of
// one 2048-wide layer, 11 + 26 for 4096 of the seven 4B-sized at r = 64)
struct XqFinishExtDev { XqDev q; uint32_t fx, blocks; ExtDev ext; };
static_assert(sizeof(KBatch<XqFinishExtDev>) <= 4096, "kernel arguments");
template <int CAP>
__global__ __launch_bounds__(256) void xq_finish_ext_kernel(const KBatch<XqFinishExtDev, CAP> tb, int rp) {
    uint32_t bx, by;
    const XqFinishExtDev& a = tb.a[kbatch_find(tb, bx, by)];
    if (bx < a.blocks) xq_finish_body(a.q, rp, bx % a.fx, bx / a.fx);
    else ext_prep_body(a.ext, (int64_t)(bx - a.blocks) * 256 + threadIdx.x);
}

// ---------------------------------------------------------------------------
// xq for one column (the paper's rank) and few tokens: on the vector units, from the fp32 column itself.  A lane multiplies eight
// consecutive values of four tokens with the values of Q that belong to them (fp32 products and sums, a lane's in order, then lanes and
// waves pairwise: fewer roundings than a sum over d_in of three planes); the waves of a workgroup share d_in in chunks of 512, as many
// as it has, and tokens otherwise.  The kernels above pad Q to 16 columns of three planes, and few tokens leave them to share d_in
// among workgroups, whose sums take a launch of their own: 432 tokens of a 1024-wide layer 5.1 + 3.1 us there and 4.4 here.  For four columns
// (the rows of Q are then twice the bytes of the four tokens) a step is 0 to 12 % slower this way.
// The line at 8192 tokens is a cautious one: of a lone layer's basis (K = 3, us with the planes, this way) it keeps out 92 and 83 at 512
// wide, 147 and 127 at 4096, 308 and 256 at 12288 on 8192 tokens, and 109 and 101, 203 and 194, 578 and 557 on 16384; below it, 512 to 12288
// wide, it lets in 72 and 59 to 96 and 75 on 432 tokens and 93 and 83 to 278 and 255 on 8064.  Errors against 64 bits are the same to 5 %
// or smaller (385 tokens of 2048: 4.6e-8 and 4.5e-8; 432 of 1024: 4.1e-8 and 3.4e-8).  The waves that share d_in: one, two and four of them 59, 58
// and 59 at 512 wide on 432 tokens (79, 80 and 83 on 6144), 65, 62 and 62 at 2560, 90, 80 and 74 at 12288
// ---------------------------------------------------------------------------
constexpr int XQN_TOK = 4, XQN_CHUNK = 512;
bool xq_narrow(int64_t M, int64_t K, int r) { return r == 1 && M < 8192 && K >= 8; }
struct XqNarrowDev {
    const bf16_t* X; const float* Q; int64_t ldx, M, K, m_pad;
    float* T; bf16_t* TpackT; bf16_t* Xext;
    int kw, vec;                 // waves that share d_in; 16-byte loads of Q
    const double* norm2; int norm_blocks; int* flag;
    const float* splits; int nsplit;
};
// A column of partial sums that every workgroup adds up for itself, instead of a launch that does: up to 16 loads a thread, 32 for one or two rows of
// the column each.  A lone layer's basis (K = 3) with that launch and so, us: 256 wide on 100 tokens 37.2 and 32.8, on 2048 51.8 and 41.2; 512 on 2048 51.5
// and 47.1; 1024 on 432 41.9 and 39.9.  Beyond the lines: 1024 on 1000 (two turns of loads) 45.0 and 46.1, on 2000 (four) 52.5 and 58.6; 2048 on 100
// 40.6 and 41.5, on 256 41.9 and 43.0.  Many layers at once (686 workgroups, where the sums wait for each other) 12 a launch and 19.5, for a launch
// less: a product alone in its launch, of a workgroup a compute unit at most
constexpr int XQN_SUM_ROWS = 1024;
static int xqn_waves(int64_t K) { return K > 3 * XQN_CHUNK ? 4 : K > XQN_CHUNK ? 2 : 1; }
bool xq_sums_column(int64_t M, int64_t K, int nsplit) {
    return K <= XQN_SUM_ROWS && (K + 255) / 256 * nsplit <= (K <= 512 ? 32 : 16) && M * xqn_waves(K) <= 256 * 4 * XQN_TOK;
}

template <bool SUMS>
__device__ __forceinline__ void xq_narrow_body(const XqNarrowDev& a, uint32_t bx) {
    constexpr int U = 2;                                        // chunks in flight
    __shared__ float part[4][XQN_TOK];
    __shared__ __align__(16) float column[SUMS ? XQN_SUM_ROWS : 4];
    __shared__ double norms[SUMS ? XQN_SUM_ROWS / 256 : 1][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = a.kw, wk = wave % kw, wt = wave / kw;
    const int64_t K = a.K, tw = ((int64_t)bx * (4 / kw) + wt) * XQN_TOK;        // the wave's first token
    const bf16_t* xr[XQN_TOK];
#pragma unroll
    for (int t = 0; t < XQN_TOK; ++t) xr[t] = a.X + min(tw + t, a.M - 1) * a.ldx;
    // A column that is still to be normalised: the result is, in fp64, as the columns between power steps are by qr1_scale_kernel.  The
    // column is X^T T of the step before, of size |X|^2, and multiplied as it stands would make sums of size |X|^3: it is read times the
    // power of two that brings its norm to [1, 2), which is exact, so the bits are the same wherever such sums are normal numbers
    double scale = 1.0;                        // (set in the waves that have a chunk: wave 0, which writes the results, among them)
    int down = 0;
    float acc[XQN_TOK] = {};
    const int64_t nchunk = (K + XQN_CHUNK - 1) / XQN_CHUNK;
    for (int64_t c0 = wk; c0 < nchunk; c0 += kw * U) {
        // (never conditional on the lane: what lies past the end, in whole eights, is read from the last place and left out)
        uint4 x[U][XQN_TOK];
        float q[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = min((c0 + u * kw) * XQN_CHUNK + 8 * lane, K - 8);
#pragma unroll
            for (int t = 0; t < XQN_TOK; ++t) x[u][t] = *reinterpret_cast<const uint4*>(xr[t] + k);
            if constexpr (SUMS) continue;
            const float* src = a.Q + k;
            if (a.vec) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const float4 v = reinterpret_cast<const float4*>(src)[i];
                    q[u][4 * i] = v.x; q[u][4 * i + 1] = v.y; q[u][4 * i + 2] = v.z; q[u][4 * i + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) q[u][i] = src[i];
            }
        }
        if (SUMS && c0 == wk) {                     // (every wave has a chunk: all of them are here together)
            const int rows = (int)K, nsplit = a.nsplit, blocks = (rows + 255) / 256, loads = blocks * nsplit;
            double sum = 0.0;
            int ls = 0, lrow = tid, s = 0, row = tid;
            for (int e0 = 0; e0 < loads; e0 += 16) {                // (uniform)
                float v[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    v[e] = e0 + e < loads ? a.splits[ls * rows + min(lrow, rows - 1)] : 0.f;
                    if (++ls == nsplit) { ls = 0; lrow += 256; }
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    if (e0 + e >= loads) break;
                    sum += (double)v[e];
                    if (++s == nsplit) {
                        column[row] = row < rows ? (float)sum : 0.f;
                        sum = 0.0; s = 0; row += 256;
                    }
                }
            }
            // the squared norm as qr1_sumsq_kernel and the branch above add it up; four blocks of 256 rows side by side (of those past the end
            // nothing is used)
            for (int b0 = 0; b0 < blocks; b0 += 4) {
                double ss[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) ss[b] = (double)column[(b0 + b) * 256 + tid] * (double)column[(b0 + b) * 256 + tid];
#pragma unroll
                for (int off = 32; off > 0; off >>= 1)
#pragma unroll
                    for (int b = 0; b < 4; ++b) ss[b] += __shfl_xor(ss[b], off);
                if (lane == 0)
#pragma unroll
                    for (int b = 0; b < 4; ++b) norms[b0 + b][wave] = ss[b];
            }
            __syncthreads();
            for (int b = 0; b < blocks; ++b) sum += (norms[b][0] + norms[b][1]) + (norms[b][2] + norms[b][3]);
            if (!(sum > 0.0)) {
                if (tid == 0 && bx == 0) *a.flag = 1;
                sum = 1.0;
            }
            down = ((__double2hiint(sum) >> 20) - 1023) >> 1;
            scale = ldexp(1.0 / sqrt(sum), down);
        }
        if constexpr (SUMS)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = (int)min((c0 + u * kw) * XQN_CHUNK + 8 * lane, K - 8);
#pragma unroll
                for (int i = 0; i < 8; ++i) q[u][i] = column[k + i];
            }
        if (!SUMS && a.norm2 != nullptr && c0 == wk) {                      // (behind the first chunks' loads: ahead of them the bases of 12288-wide layers take 1 to 4 % longer)
            double sum = 0.0;
            for (int b0 = 0; b0 < a.norm_blocks; b0 += 16) {       // uniform: every thread adds the same values
                double v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = b0 + i < a.norm_blocks ? a.norm2[b0 + i] : 0.0;
#pragma unroll
                for (int i = 0; i < 16; ++i) sum += v[i];
            }
            if (!(sum > 0.0)) {
                if (tid == 0 && bx == 0) *a.flag = 1;
                sum = 1.0;
            }
            down = ((__double2hiint(sum) >> 20) - 1023) >> 1;      // (squares of fp32 values: never subnormal)
            scale = ldexp(1.0 / sqrt(sum), down);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if ((c0 + u * kw) * XQN_CHUNK + 8 * lane >= K) continue;
#pragma unroll
            for (int i = 0; i < 8; ++i) q[u][i] = ldexpf(q[u][i], -down);
#pragma unroll
            for (int t = 0; t < XQN_TOK; ++t) {
                const uint32_t w[4] = {x[u][t].x, x[u][t].y, x[u][t].z, x[u][t].w};
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[t] = fmaf(__uint_as_float((e & 1) ? w[e >> 1] & 0xFFFF0000u : w[e >> 1] << 16), q[u][e], acc[t]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < XQN_TOK; ++t) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc[t] += __shfl_xor(acc[t], off);
        if (lane == 0) part[wave][t] = acc[t];
    }
    __syncthreads();
    // a thread four tokens and a column of the outputs' sixteen: all but the first are zero
    const int g = tid >> 4, k = tid & 15;
    if (g >= 4 / kw) return;
    floatx4 v = {0.f, 0.f, 0.f, 0.f};
    if (k == 0) {
#pragma unroll
        for (int t = 0; t < XQN_TOK; ++t) {
            v[t] = part[g * kw][t];
            if (kw == 2) v[t] += part[g * kw + 1][t];
            if (kw == 4) v[t] = (v[t] + part[1][t]) + (part[2][t] + part[3][t]);
            v[t] = (float)((double)v[t] * scale);
        }
    }
    xq_emit(v, a.M, 1, 16, a.T, a.TpackT, a.m_pad, a.Xext, ((int64_t)bx * (4 / kw) + g) * XQN_TOK, k);
}
template <int CAP, bool SUMS>
__global__ __launch_bounds__(256) void xq_narrow_many_kernel(const KBatch<XqNarrowDev, CAP> tb) {
    uint32_t bx, by;
    const XqNarrowDev& a = tb.a[kbatch_find(tb, bx, by)];
    xq_narrow_body<SUMS>(a, bx);
}
// with the W sides of forwards' extension operands
struct XqNarrowExtDev { XqNarrowDev q; uint32_t blocks; ExtDev ext; };
static_assert(sizeof(KBatch<XqNarrowExtDev>) <= 4096, "kernel arguments");
template <int CAP>
__global__ __launch_bounds__(256) void xq_narrow_ext_kernel(const KBatch<XqNarrowExtDev, CAP> tb) {
    uint32_t bx, by;
    const XqNarrowExtDev& a = tb.a[kbatch_find(tb, bx, by)];
    if (bx < a.blocks) xq_narrow_body<false>(a.q, bx);
    else ext_prep_body(a.ext, (int64_t)(bx - a.blocks) * 256 + threadIdx.x);
}

static XqNarrowDev xqn_dev(const XqArgs& a, uint64_t& workgroups) {
    XqNarrowDev d{a.X, a.Q, a.ldx, a.M, a.K, a.m_pad, a.T, a.TpackT, a.Xext, xqn_waves(a.K), (reinterpret_cast<uintptr_t>(a.Q) & 15) == 0,
                  a.norm2, a.norm_blocks, a.flag, a.splits, a.nsplit};
    const int64_t tok = XQN_TOK * (4 / d.kw);
    workgroups = (uint64_t)(((a.TpackT ? a.m_pad : a.M) + tok - 1) / tok);
    return d;
}
static hipError_t launch_xq_narrow(const XqArgs* const* a, int n, hipStream_t st) {
    KBatch<XqNarrowDev> tb;
    KBatch<XqNarrowExtDev> eb;
    tb.n = eb.n = 0;
    uint64_t blocks = 0, eblocks = 0;
    for (int i = 0; i < n; ++i) {
        uint64_t wgs, ext_wgs = 0;
        const XqNarrowDev d = xqn_dev(*a[i], wgs);
        if (!a[i]->ext) {
            tb.first[tb.n] = (uint32_t)blocks;
            tb.gx[tb.n] = (uint32_t)wgs;
            tb.a[tb.n++] = d;
            blocks += wgs;
        } else {
            const ExtDev e = ext_dev(*a[i]->ext, ext_wgs);
            eb.first[eb.n] = (uint32_t)eblocks;
            eb.gx[eb.n] = (uint32_t)(wgs + ext_wgs);
            eb.a[eb.n++] = XqNarrowExtDev{d, (uint32_t)wgs, e};
            eblocks += wgs + ext_wgs;
        }
        if (blocks > 0x7FFFFFFFull || eblocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    }
    if (tb.n == 1 && tb.a[0].splits) hipLaunchKernelGGL((xq_narrow_many_kernel<1, true>), dim3((unsigned)blocks), dim3(256), 0, st, kbatch_one(tb));
    else if (tb.n == 1) hipLaunchKernelGGL((xq_narrow_many_kernel<1, false>), dim3((unsigned)blocks), dim3(256), 0, st, kbatch_one(tb));
    else if (tb.n > 1) hipLaunchKernelGGL((xq_narrow_many_kernel<kBatchMax, false>), dim3((unsigned)blocks), dim3(256), 0, st, tb);
    const hipError_t err = tb.n > 0 ? hipGetLastError() : hipSuccess;
    if (err != hipSuccess || eb.n == 0) return err;
    if (eb.n == 1) hipLaunchKernelGGL(xq_narrow_ext_kernel<1>, dim3((unsigned)eblocks), dim3(256), 0, st, kbatch_one(eb));
    else hipLaunchKernelGGL(xq_narrow_ext_kernel<kBatchMax>, dim3((unsigned)eblocks), dim3(256), 0, st, eb);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The projection P = X B of a perturbed forward (up to 16 columns) and the W side of its extension operands in one launch, from B as it
// is: a model's program makes this chain once per linear layer and sign.  A workgroup has 32 tokens, its eight waves share d_in in
// 64-wide slices, and nothing goes through LDS but the eight sums: a lane asks for its 16-byte chunks of X (two tokens, a line each)
// and for sixteen values of its column of B, splits these into the planes and multiplies; two slices in flight.  Products and sums are
// those of xq_bf16_many_kernel, the sums over d_in in eight parts that are added in order.
// Bound by what a compute unit takes in, some 60 GB/s: a workgroup's rows of X and as many bytes of B.  (Three and four slices in flight, B in
// 16-byte pieces through LDS, sixteen waves, another order of the chunks: the same time or 5 to 30 % more.)  With the planes of B and the
// W side in a launch ahead, which is bound by its latency, and the projection in workgroups of 64 tokens it took, r = 16, us: 4.8 + 10.5
// at 8192 x 2048 -> 2048 and 10.0 so; 4.8 + 44 at 8192 x 6144 and 33; 4.8 + 5 + 4.5 (shares of d_in, added by a third launch) at 385 x 2048
// and 8.5.  A decoder on 8192 tokens 15345 a step and 14988, on 385 1931 and 1834
// ---------------------------------------------------------------------------
constexpr int XQE_TOK = 32, XQE_WAVES = 8;
struct XqExtDev {
    const bf16_t* X; const float* B; int64_t ldx, M, K; int r;
    float* T; bf16_t* Xext;
};
__device__ __forceinline__ void xq_ext_body(const XqExtDev& a, uint32_t bx) {
    __shared__ float part[XQE_WAVES][XQE_TOK][17];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15, lg = lane >> 4, r = a.r;
    const int64_t K = a.K, t0 = (int64_t)bx * XQE_TOK;
    const bf16_t* xr[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) xr[m] = a.X + min(t0 + m * 16 + lm, a.M - 1) * a.ldx;
    const float* bc = a.B + min(lm, r - 1);
    const bool col = lm < r;
    struct Slice { uint4 x[2][2]; float b[2][8]; };
    // lane (lm, lg): 16-byte chunks 2 lg and 2 lg + 1 of a row's slice, and column lm of the rows of B that belong to them.  (Never
    // conditional on the lane: what lies past the end, in whole eights, is read from the last place and left out)
    auto load = [&](Slice& s, int64_t slice) __attribute__((always_inline)) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const int64_t k = min(slice * XQ_BK + lg * 16 + sub * 8, K - 8);
#pragma unroll
            for (int m = 0; m < 2; ++m) s.x[m][sub] = *reinterpret_cast<const uint4*>(xr[m] + k);
            const float* src = bc + k * r;
#pragma unroll
            for (int j = 0; j < 8; ++j) s.b[sub][j] = src[j * r];
        }
    };
    floatx4 acc[2] = {};
    auto multiply = [&](const Slice& s, int64_t slice) __attribute__((always_inline)) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const bool in = slice * XQ_BK + lg * 16 + sub * 8 < K;
            Frag x[2], q[3];
#pragma unroll
            for (int m = 0; m < 2; ++m) x[m].u = in ? s.x[m][sub] : make_uint4(0, 0, 0, 0);
            uint32_t w[3][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float v0 = in && col ? s.b[sub][2 * j] : 0.f, v1 = in && col ? s.b[sub][2 * j + 1] : 0.f;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) {
                    w[pl][j] = pack_bf16x2(v0, v1);
                    v0 -= __uint_as_float(w[pl][j] << 16);
                    v1 -= __uint_as_float(w[pl][j] & 0xFFFF0000u);
                }
            }
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) q[pl].u = make_uint4(w[pl][0], w[pl][1], w[pl][2], w[pl][3]);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[m].v, q[pl].v, acc[m], 0, 0, 0);
        }
    };
    const int64_t slices = (K + XQ_BK - 1) / XQ_BK;
    Slice s0, s1;
    load(s0, wave);
    for (int64_t sl = wave; sl < slices; sl += 2 * XQE_WAVES) {
        load(s1, sl + XQE_WAVES);
        multiply(s0, sl);
        load(s0, sl + 2 * XQE_WAVES);
        multiply(s1, sl + XQE_WAVES);          // (behind the last slice: nothing that counts)
    }
    // D layout: row (token) = 4 lg + e, column lm
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[wave][m * 16 + lg * 4 + e][lm] = acc[m][e];
    __syncthreads();
    const int k = tid & 15, tok = tid >> 4;
    float v = part[0][tok][k];
#pragma unroll
    for (int w = 1; w < XQE_WAVES; ++w) v += part[w][tok][k];
    const int64_t t = t0 + tok;
    if (t >= a.M) return;
    if (k >= r) v = 0.f;
    if (a.T != nullptr && k < r) a.T[t * r + k] = v;
    if (a.Xext != nullptr) store_ext(a.Xext, t, k, 16, v);
}
static_assert(XQE_TOK * 16 == XQE_WAVES * 64, "a thread a value");
__global__ __launch_bounds__(64 * XQE_WAVES) void xq_ext_kernel(const XqExtDev a, uint32_t blocks, const ExtDev ext) {
    if (blockIdx.x < blocks) xq_ext_body(a, blockIdx.x);
    else ext_prep_body(ext, (int64_t)(blockIdx.x - blocks) * (64 * XQE_WAVES) + threadIdx.x);
}
// One round of workgroups, and no more of d_in to a workgroup than the tokens make up for: few workgroups that take in all of a wide layer's d_in each
// are slower than shares of d_in and a launch that adds them, and more workgroups than compute units slower than the 64-token ones of
// xq_bf16_many_kernel.  A perturbed forward to 384 outputs, r = 16, us, those launches and this one: 385 tokens of 2048 20.8 and 18.6, of 3072
// 22.4 and 22.0, of 4096 23.4 and 25.2, of 6144 27.0 and 32.6; 3001 of 2560 28.5 and 27.4, of 4096 31.8 and 31.4, of 6144 38.1 and 40.3; 6000
// of 5120 54.9 and 52.0, 8192 of 2048 30.0 and 25.5, of 6144 66.7 and 59.4, of 8192 82.7 and 85.5; 9000 of 512 17.1 and 18.0, of 2048 30.8 and
// 32.1, of 6144 69.4 and 76.3, 16384 of 4096 76.9 and 75.5, of 8192 171 and 188.  On this side of the line d_in has fewer than eight shares
// there, so the sums here are the more exact ones (8192 of 6144: 3.1e-7 of the result against 8.6e-7; beyond it, 385 of 6144 in sixteen shares,
// it was 3.0e-7 against 2.5e-7)
constexpr int XQE_CUS = 256;
bool xq_ext_ok(int64_t M, int64_t K, int r) { return r <= 16 && K >= 8 && M <= (int64_t)XQE_CUS * XQE_TOK && (K <= 2048 || M >= K + K / 8); }
hipError_t launch_xq_ext(const XqArgs& a, const GemmExtArgs* ext, hipStream_t st) {
    if (!xq_ext_ok(a.M, a.K, a.r) || !a.Q || a.TpackT || (ext && (ext->planes || ext->P))) return hipErrorInvalidValue;
    const uint64_t wgs = (uint64_t)((a.M + XQE_TOK - 1) / XQE_TOK);
    uint64_t ext_wgs = 0;
    ExtDev e{};
    if (ext) e = ext_dev(*ext, ext_wgs, 64 * XQE_WAVES);
    if (wgs + ext_wgs > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (wgs + ext_wgs == 0) return hipSuccess;
    const XqExtDev d{a.X, a.Q, a.ldx, a.M, a.K, a.r, a.T, a.Xext};
    hipLaunchKernelGGL(xq_ext_kernel, dim3((unsigned)(wgs + ext_wgs)), dim3(64 * XQE_WAVES), 0, st, d, (uint32_t)wgs, e);
    return hipGetLastError();
}

// number of d_in splits for M tokens (1 = the token blocks alone fill the chip, or d_in is too short to share)
static int xq_splits(int64_t rows, int64_t K) {
    const int64_t blocks = (rows + XQ_TOK - 1) / XQ_TOK;
    const int64_t slices = K / XQ_BK;
    if (blocks >= 128 || slices < 16) return 1;
    int64_t want = 256 / blocks;
    if (want > slices / 8) want = slices / 8;      // at least eight slices each: the depth of the load ring
    if (want > 16) want = 16;
    return (int)(want < 1 ? 1 : want);
}

size_t xq_part_bytes(int64_t M, int64_t K, int rp) {
    const int64_t m_pad = (M + 31) / 32 * 32;
    const int ns = xq_splits(m_pad, K);
    return ns > 1 ? (size_t)ns * m_pad * rp * sizeof(float) : 0;
}

template <int NB, int DEEP, int CAP>
static hipError_t launch_xq_ring(const KBatch<XqDev, CAP>& tb, unsigned blocks, hipStream_t st) {
    const int smem = XqRing<NB, DEEP>::STAGES * xq_slot_bytes(NB);
    static bool set = false;
    if (!set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(xq_bf16_many_kernel<NB, DEEP, CAP>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL((xq_bf16_many_kernel<NB, DEEP, CAP>), dim3(blocks), dim3(256), smem, st, tb);
    return hipGetLastError();
}
template <int NB, int MB, int CAP>
static hipError_t launch_xq_direct(const KBatch<XqDev, CAP>& tb, unsigned blocks, hipStream_t st) {
    const int smem = XQD_STAGES * xqd_loads(NB) * 4096;
    static bool set = false;
    if (!set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(xq_direct_many_kernel<NB, MB, CAP>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL((xq_direct_many_kernel<NB, MB, CAP>), dim3(blocks), dim3(256), smem, st, tb);
    return hipGetLastError();
}
// (the result depends neither on the ring's depth nor on the tokens of a workgroup: same slices, same order)
template <int NB, int CAP>
static hipError_t launch_xq_many_nb(const KBatch<XqDev, CAP>& tb, unsigned blocks, int mb, bool half_cu, hipStream_t st) {
    if constexpr (NB >= 3) return mb == 2 ? launch_xq_direct<NB, 2>(tb, blocks, st) : launch_xq_direct<NB, 1>(tb, blocks, st);
    else if (half_cu) return launch_xq_ring<NB, 2>(tb, blocks, st);
    else return blocks >= 512 ? launch_xq_ring<NB, 0>(tb, blocks, st) : launch_xq_ring<NB, 1>(tb, blocks, st);
}

template <int CAP>
static hipError_t launch_xq_cap(const KBatch<XqDev, CAP>& tb, unsigned blocks, int rp, int mb, bool half_cu, hipStream_t st) {
    switch (rp / 16) {
        case 1: return launch_xq_many_nb<1>(tb, blocks, mb, half_cu, st);
        case 2: return launch_xq_many_nb<2>(tb, blocks, mb, half_cu, st);
        case 3: return launch_xq_many_nb<3>(tb, blocks, mb, half_cu, st);
        case 4: return launch_xq_many_nb<4>(tb, blocks, mb, half_cu, st);
        default: return hipErrorInvalidValue;
    }
}

template <int MB, bool HALF_CU>
static hipError_t launch_xq_group(const KBatch<XqGroupDev>& tb, unsigned blocks, int most, hipStream_t st) {
    static bool set = false;
    if (!set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(xq_group_kernel<MB, HALF_CU>), hipFuncAttributeMaxDynamicSharedMemorySize, xq_group_smem<HALF_CU>(kXShare));
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL((xq_group_kernel<MB, HALF_CU>), dim3(blocks), dim3(256), xq_group_smem<HALF_CU>(most), st, tb);
    return hipGetLastError();
}
// the products of a launch in groups that share X: *done = false where there are none (or not up to 16 columns)
static hipError_t launch_xq_groups(const KBatch<XqDev>& tb, int rp, bool half_cu, hipStream_t st, bool* done) {
    *done = false;
    if (rp != 16) return hipSuccess;
    KBatch<XqGroupDev> gr;
    gr.n = 0;
    int most = 1;
    int64_t widest = 0;                        // of those that share
    uint64_t half = 0;                         // workgroups of 128 tokens
    for (int i = 0; i < tb.n; ++i) {
        const XqDev& p = tb.a[i];
        int g = 0;
        for (; g < gr.n; ++g) {
            const XqGroupDev& d = gr.a[g];
            if (d.nb < kXShare && d.X == p.X && d.ldx == p.ldx && d.M == p.M && d.K == p.K && d.m_pad == p.m_pad && d.ns == p.ns && (d.TpackT[0] != nullptr) == (p.TpackT != nullptr)) break;
        }
        XqGroupDev& d = gr.a[g];
        if (g == gr.n) {
            d.X = p.X; d.ldx = p.ldx; d.M = p.M; d.K = p.K; d.m_pad = p.m_pad; d.ns = p.ns; d.nb = 0;
            gr.n++;
            half += (uint64_t)((p.M + 2 * XQ_TOK - 1) / (2 * XQ_TOK)) * (uint64_t)p.ns;
        }
        d.Qpack[d.nb] = p.Qpack; d.T[d.nb] = p.T; d.TpackT[d.nb] = p.TpackT; d.part[d.nb] = p.part; d.Xext[d.nb] = p.Xext; d.r[d.nb] = p.r;
        if (++d.nb > 1) widest = std::max(widest, d.K);
        most = std::max(most, d.nb);
    }
    if (most == 1) return hipSuccess;
    // Workgroups of 128 tokens read the planes half as often, but are fewer and longer: us a launch of all products of the 8B-sized layers on 16384
    // tokens (beside their forwards) 524 with 64 tokens and 482 with 128, of 2.3 decoder layers (2048 wide) on 8192 109 and 116, 4B-sized (2560) on
    // 3001 51.2 and 52.4
    const int mb = half >= 256 && widest >= 4096 ? 2 : 1;
    uint64_t blocks = 0;                       // (deepest first, as the products came)
    for (int g = 0; g < gr.n; ++g) {
        const int64_t rows = gr.a[g].TpackT[0] ? gr.a[g].m_pad : gr.a[g].M;
        gr.first[g] = (uint32_t)blocks;
        const int tok = gr.a[g].nb == 1 ? XQ_TOK : mb * XQ_TOK;
        gr.gx[g] = (uint32_t)((rows + tok - 1) / tok);
        blocks += (uint64_t)gr.gx[g] * (uint32_t)gr.a[g].ns;
    }
    if (blocks < XQ_GROUP_MIN) return hipSuccess;
    const unsigned grid = (unsigned)blocks;
    const hipError_t e = half_cu ? (mb == 2 ? launch_xq_group<2, true>(gr, grid, most, st) : launch_xq_group<1, true>(gr, grid, most, st))
                                 : (mb == 2 ? launch_xq_group<2, false>(gr, grid, most, st) : launch_xq_group<1, false>(gr, grid, most, st));
    *done = true;
    return e;
}

hipError_t launch_xq_bf16_many(const XqArgs* a, int n, bool half_cu, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    int rp = 0;
    uint64_t half = 0;                         // workgroups of 128 tokens
    // the deepest workgroups first, so that the launch does not end on a few of them (a share of d_in is not deep because d_in is: 1879 tokens
    // of layers 584, 824 and 3648 wide, the last in seven shares, r = 8, three launches 50 us by d_in and 44 so)
    int order[kBatchMax], count = 0;
    int64_t depth[kBatchMax];
    const XqArgs* narrow[kBatchMax];
    int n_narrow = 0;
    for (int m = 0; m < n; ++m) {
        if (a[m].M == 0) continue;
        if (rp == 0) rp = a[m].rp;
        if (a[m].rp != rp || a[m].m_pad % 4 || (a[m].ext && (a[m].ext->planes || a[m].ext->P))) return hipErrorInvalidValue;       // one padded rank per launch
        if (xq_narrow(a[m].M, a[m].K, a[m].r)) {
            if (a[m].splits ? n > 1 || a[m].ext || !xq_sums_column(a[m].M, a[m].K, a[m].nsplit) : !a[m].Q) return hipErrorInvalidValue;
            narrow[n_narrow++] = &a[m];
            continue;
        }
        const int ns = a[m].part ? xq_splits(a[m].m_pad, a[m].K) : 1;
        depth[m] = a[m].K / ns;
        int at = count++;
        for (; at > 0 && depth[order[at - 1]] < depth[m]; --at) order[at] = order[at - 1];
        order[at] = m;
        half += (uint64_t)((a[m].M + 2 * XQ_TOK - 1) / (2 * XQ_TOK)) * (uint64_t)ns;
    }
    const hipError_t en = launch_xq_narrow(narrow, n_narrow, st);
    if (en != hipSuccess || count == 0) return en;
    const int mb = rp >= 48 && half >= 256 ? 2 : 1;      // (where that leaves no compute unit without a workgroup)
    KBatch<XqDev> tb, fin;
    KBatch<XqFinishExtDev> fext;
    tb.n = fin.n = fext.n = 0;
    uint64_t blocks = 0, fin_blocks = 0, fext_blocks = 0;
    for (int i = 0; i < count; ++i) {
        const int m = order[i];
        XqDev d;
        d.X = a[m].X; d.ldx = a[m].ldx; d.M = a[m].M; d.K = a[m].K; d.Qpack = a[m].Qpack; d.r = a[m].r;
        d.T = a[m].T; d.TpackT = a[m].TpackT; d.m_pad = a[m].m_pad;
        d.Xext = a[m].Xext;
        d.ns = a[m].part ? xq_splits(a[m].m_pad, a[m].K) : 1;
        d.part = d.ns > 1 ? a[m].part : nullptr;
        const int64_t rows = a[m].TpackT ? a[m].m_pad : a[m].M;
        const uint32_t gx = (uint32_t)((rows + mb * XQ_TOK - 1) / (mb * XQ_TOK));
        tb.first[tb.n] = (uint32_t)blocks; tb.gx[tb.n] = gx; tb.a[tb.n++] = d;
        blocks += (uint64_t)gx * (uint32_t)d.ns;
        const int ftok = d.TpackT ? XQF_TOK : XQF_TOK_ROWS;
        const uint32_t fx = (uint32_t)((rows + ftok - 1) / ftok), fwgs = fx * (uint32_t)(rp / 16);
        if (a[m].ext) {
            uint64_t wgs;
            XqFinishExtDev& x = fext.a[fext.n];
            x.q = d; x.fx = fx; x.blocks = d.ns > 1 ? fwgs : 0;
            x.ext = ext_dev(*a[m].ext, wgs);
            wgs += x.blocks;
            if (wgs == 0) continue;
            fext.first[fext.n] = (uint32_t)fext_blocks; fext.gx[fext.n++] = (uint32_t)wgs;
            fext_blocks += wgs;
        } else if (d.ns > 1) {
            fin.first[fin.n] = (uint32_t)fin_blocks; fin.gx[fin.n] = fx; fin.a[fin.n++] = d;
            fin_blocks += fwgs;
        }
    }
    if (blocks > 0x7FFFFFFFull || fin_blocks > 0x7FFFFFFFull || fext_blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    bool shared = false;
    hipError_t e = launch_xq_groups(tb, rp, half_cu, st, &shared);
    if (e != hipSuccess) return e;
    if (!shared) e = tb.n == 1 ? launch_xq_cap(kbatch_one(tb), (unsigned)blocks, rp, mb, half_cu, st) : launch_xq_cap(tb, (unsigned)blocks, rp, mb, half_cu, st);
    if (e == hipSuccess && fext.n > 0) {
        if (fext.n == 1) hipLaunchKernelGGL(xq_finish_ext_kernel<1>, dim3((unsigned)fext_blocks), dim3(256), 0, st, kbatch_one(fext), rp);
        else hipLaunchKernelGGL(xq_finish_ext_kernel<kBatchMax>, dim3((unsigned)fext_blocks), dim3(256), 0, st, fext, rp);
        e = hipGetLastError();
    }
    if (e != hipSuccess || fin.n == 0) return e;
    const dim3 fin_grid((unsigned)fin_blocks);
    if (fin.n == 1) hipLaunchKernelGGL(xq_finish_many_kernel<1>, fin_grid, dim3(256), 0, st, kbatch_one(fin), rp);
    else hipLaunchKernelGGL(xq_finish_many_kernel<kBatchMax>, fin_grid, dim3(256), 0, st, fin, rp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// xtt: workgroup = (panel of 128 features) x (token range); its four waves take 32-token steps in turn and add their sums in LDS.
// ALONE (r > 16 only): a wave takes the four waves' steps one wave after the other: the same sums in the same order, a quarter of
// the workgroups, and no adding of 128 rows of up to 64 columns in LDS, which takes longer than the few steps it follows.
// MFMA roles: A = T^T planes (rows = k, K = tokens), B = X^T (K = tokens, cols = features).
// X is row-major in features, so a lane loads 8 features x 8 tokens as eight 16-byte rows and
// transposes them in registers (byte permutes) into eight token-contiguous operands.
// ---------------------------------------------------------------------------
constexpr int XTT_PANEL = 128;
constexpr int XTT_STEP = 32;

int xtt_num_splits(int64_t M, int64_t K) {
    const int64_t panels = (K + XTT_PANEL - 1) / XTT_PANEL;
    // at least about one workgroup per CU; with many tokens up to eight token ranges even when the panels alone fill
    // the chip (activations wider than the last-level cache come from HBM and need the bytes in flight: 814 -> 696 us
    // per extraction at 16384 x 12288); more ranges than that cost more in partial sums than they hide
    int64_t want = (256 + panels - 1) / panels;
    const int64_t by_tokens = M / 1024 < 8 ? M / 1024 : 8;
    if (want < by_tokens) want = by_tokens;
    const int64_t max_splits = (M + 4 * XTT_STEP - 1) / (4 * XTT_STEP);
    if (want > max_splits) want = max_splits;
    if (want < 1) want = 1;
    if (want > 16) want = 16;
    return (int)want;
}

// bx: panel of features, by: token range
template <int NB>
__device__ __forceinline__ void xtt_bf16_body(const bf16_t* __restrict__ X, int64_t ldx, int64_t M, int64_t K,
                                              const bf16_t* __restrict__ TpackT, int64_t m_pad,
                                              float* __restrict__ partial, int64_t tok_per_split, int one, uint32_t bx, uint32_t by) {
    constexpr int RP = NB * 16;
    extern __shared__ __align__(16) float sbuf[];   // [XTT_PANEL][RP]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lc = lane & 15, lg = lane >> 4;
    const int64_t db = (int64_t)bx * XTT_PANEL;
    const int split = (int)by;
    const int64_t ts = (int64_t)split * tok_per_split;
    const int64_t te = min(ts + tok_per_split, m_pad);

    floatx4 acc[NB][8];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[nb][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int64_t dcol = db + lc * 8;
    const int64_t dload = min(dcol, K - 8);        // (features past the end repeat the last, unstored)
    // one 32-token step: 8 KB of X and the T planes per wave.  The next step's loads are issued before this step's
    // matrix work (twice the bytes in flight: with one step in flight the sweep ran at memory latency); they are
    // unconditional, the step after the last one re-reads the last (clamped) and is dropped.
    auto load_step = [&](int64_t tb, uint4 (&v)[8], Frag (&a)[NB][3]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t t = min(tb + lg * 8 + i, M - 1);   // rows past M meet zero planes
            v[i] = *reinterpret_cast<const uint4*>(X + t * ldx + dload);
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                a[nb][pl].u = *reinterpret_cast<const uint4*>(TpackT + ((int64_t)(pl * RP + nb * 16 + lc)) * m_pad + tb + lg * 8);
    };
    constexpr int STRIDE = 4 * XTT_STEP;
    auto multiply = [&](const uint4 (&v)[8], const Frag (&a)[NB][3]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // word q of v[i] holds features 2q (low half) and 2q+1 (high half) of token i
            const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
            const int q = j >> 1;
            Frag b;
            const uint32_t* w0 = reinterpret_cast<const uint32_t*>(&v[0]);
            uint32_t o[4];
#pragma unroll
            for (int pp = 0; pp < 4; ++pp)
                o[pp] = __builtin_amdgcn_perm(w0[(2 * pp + 1) * 4 + q], w0[(2 * pp) * 4 + q], sel);
            b.u = make_uint4(o[0], o[1], o[2], o[3]);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[nb][pl].v, b.v, acc[nb][j], 0, 0, 0);
        }
    };
    // A wave's steps: every fourth of the range, from its own number on.  Two register sets in turn: moved from one to the other at
    // the end of a step, the loads would be waited for there
    int64_t tb = ts + wave * XTT_STEP;
    if (tb < te) {
        uint4 v0[8], v1[8];
        Frag a0[NB][3], a1[NB][3];
        load_step(tb, v0, a0);
        for (; tb < te; tb += 2 * STRIDE) {
            load_step(min(tb + STRIDE, te - XTT_STEP), v1, a1);
            multiply(v0, a0);
            if (tb + STRIDE >= te) break;
            load_step(min(tb + 2 * STRIDE, te - XTT_STEP), v0, a0);
            multiply(v1, a1);
        }
    }
    // D layout: row (k within block) = 4*(lane/16) + e, col = lane%16 -> feature db + 8*lc + j
    if (NB == 1 && one) {
        // the first column alone: the waves' sums side by side, added in the same order
        if (lg == 0)
#pragma unroll
            for (int j = 0; j < 8; ++j) sbuf[wave * XTT_PANEL + lc * 8 + j] = acc[0][j][0];
        __syncthreads();
        if (tid < XTT_PANEL && db + tid < K)
            partial[(int64_t)split * K + db + tid] = ((sbuf[tid] + sbuf[XTT_PANEL + tid]) + sbuf[2 * XTT_PANEL + tid]) + sbuf[3 * XTT_PANEL + tid];
        return;
    }
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float* dst = &sbuf[(lc * 8 + j) * RP + nb * 16 + lg * 4 + e];
                        if (w == 0) *dst = acc[nb][j][e]; else *dst += acc[nb][j][e];
                    }
        }
        __syncthreads();
    }
    float* out = partial + ((int64_t)split * K + db) * RP;
    const int64_t nvalid = min((int64_t)XTT_PANEL, K - db) * RP;
    for (int idx = tid; idx < XTT_PANEL * RP; idx += 256)
        if (idx < nvalid) out[idx] = sbuf[idx];
}

// ALONE: a workgroup is four panels of one token range.  The planes of a step are the same for all of them (from memory to each wave, at
// r = 64 they were 12 KB a step against 8 KB of X) and come through LDS, X with them, two steps ahead.  A wave has 16 columns of a
// panel, 32 at r > 48: two or three waves to a SIMD, one of which multiplies while the others read, and accumulators and the sums of
// finished shares that fit the registers without moves (a wave with all 64 columns spent 330 of a step's instructions on those).
// 4096 tokens of seven 4B-sized layers: 70 -> 52 us at r = 32, 103 -> 66 at 48, 130 -> 75 at 64
template <int NB>
struct XttAlone {
    static constexpr int NBW = NB == 4 ? 2 : 1, WAVES = 4 * NB / NBW;                                      // column blocks of a wave
    static constexpr int LOADS = (3 * NB + WAVES - 1) / WAVES, XLOADS = (32 + WAVES - 1) / WAVES;        // a wave's direct loads of a step
    static constexpr int STAGE = (LOADS * WAVES + 32) * 1024;
};
template <int NB>
__device__ __forceinline__ void xtt_alone_body(const bf16_t* __restrict__ X, int64_t ldx, int64_t M, int64_t K,
                                               const bf16_t* __restrict__ TpackT, int64_t m_pad,
                                               float* __restrict__ partial, int64_t tok_per_split, uint32_t bx, uint32_t by) {
    typedef XttAlone<NB> S;
    constexpr int RP = NB * 16, SEGS = 3 * NB, NBW = S::NBW;  // 16-row segments of the planes: a direct load each, 1 KiB
    constexpr int WAVES = S::WAVES, LOADS = S::LOADS, XLOADS = S::XLOADS, STAGE = S::STAGE, X_AT = LOADS * WAVES * 1024;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) char xtt_smem[];          // [3 stages]: [segments][16 rows][32 tokens], [4 panels][32 tokens][128 features]
    typedef __attribute__((address_space(3))) void* lptr_t;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 15, lg = lane >> 4, panel = wave & 3, nb0 = (wave >> 2) * NBW;
    const int split = (int)by;
    const int64_t ts = (int64_t)split * tok_per_split, te = min(ts + tok_per_split, m_pad);
    const int64_t dcol = ((int64_t)bx * 4 + panel) * XTT_PANEL + lc * 8;
    // (features past the end repeat the last, unstored)
    const bf16_t* xcol = X + min(((int64_t)bx * 4 + panel) * XTT_PANEL + lc * 8, K - 8);

    // this wave's segments of a step: segment wave + WAVES i (past the last: the last once more, into rows nobody reads)
    const bf16_t* tsrc[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) tsrc[i] = TpackT + (int64_t)(16 * min(wave + WAVES * i, SEGS - 1) + (lane >> 2)) * m_pad + (lane & 3) * 8;

    // the step behind that at tb, of share w: the shares are every fourth step, taken one share after the other
    auto next = [&](int64_t& tb, int& w) __attribute__((always_inline)) {
        tb += 4 * XTT_STEP;
        if (tb >= te) tb = ++w < 4 ? ts + w * XTT_STEP : te;
    };
    auto issue = [&](int set, int64_t tb) __attribute__((always_inline)) {
        tb = min(tb, te - XTT_STEP);                          // (past the last step: that once more)
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(tsrc[i] + tb), (lptr_t)(xtt_smem + set * STAGE + (wave + WAVES * i) * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < XLOADS; ++i) {                    // (rows past M meet zero planes)
            const int q = min((wave >> 2) * XLOADS + i, 7);       // (three waves to a panel: the last once more)
            __builtin_amdgcn_global_load_lds((gptr_t)(xcol + min(tb + 4 * q + lg, M - 1) * ldx), (lptr_t)(xtt_smem + set * STAGE + X_AT + panel * 8192 + q * 1024), 16, 0, 0);
        }
    };
    floatx4 acc[NBW][8], tot[NBW][8];
    auto multiply = [&](int set) __attribute__((always_inline)) {
        u32x4 a[NBW][3], x[8];
        const uint32_t addr = (uint32_t)(uintptr_t)(lptr_t)(xtt_smem + set * STAGE + nb0 * 1024 + lc * 64 + lg * 16);
        const uint32_t xaddr = (uint32_t)(uintptr_t)(lptr_t)(xtt_smem + set * STAGE + X_AT + panel * 8192 + lg * 2048 + lc * 16);
        if constexpr (NB == 2)
            asm volatile("ds_read_b128 %0, %11\n\tds_read_b128 %1, %11 offset:2048\n\tds_read_b128 %2, %11 offset:4096\n\t"
                                     "ds_read_b128 %3, %12\n\tds_read_b128 %4, %12 offset:256\n\tds_read_b128 %5, %12 offset:512\n\t"
                                     "ds_read_b128 %6, %12 offset:768\n\tds_read_b128 %7, %12 offset:1024\n\tds_read_b128 %8, %12 offset:1280\n\t"
                                     "ds_read_b128 %9, %12 offset:1536\n\tds_read_b128 %10, %12 offset:1792\n\ts_waitcnt lgkmcnt(0)"
                                     : "=&v"(a[0][0]), "=&v"(a[0][1]), "=&v"(a[0][2]), "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]),
                                       "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
                                     : "v"(addr), "v"(xaddr) : "memory");
        else if constexpr (NB == 3)
            asm volatile("ds_read_b128 %0, %11\n\tds_read_b128 %1, %11 offset:3072\n\tds_read_b128 %2, %11 offset:6144\n\t"
                                     "ds_read_b128 %3, %12\n\tds_read_b128 %4, %12 offset:256\n\tds_read_b128 %5, %12 offset:512\n\t"
                                     "ds_read_b128 %6, %12 offset:768\n\tds_read_b128 %7, %12 offset:1024\n\tds_read_b128 %8, %12 offset:1280\n\t"
                                     "ds_read_b128 %9, %12 offset:1536\n\tds_read_b128 %10, %12 offset:1792\n\ts_waitcnt lgkmcnt(0)"
                                     : "=&v"(a[0][0]), "=&v"(a[0][1]), "=&v"(a[0][2]), "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]),
                                       "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
                                     : "v"(addr), "v"(xaddr) : "memory");
        else
            asm volatile("ds_read_b128 %0, %14\n\tds_read_b128 %1, %14 offset:1024\n\tds_read_b128 %2, %14 offset:4096\n\t"
                                     "ds_read_b128 %3, %14 offset:5120\n\tds_read_b128 %4, %14 offset:8192\n\tds_read_b128 %5, %14 offset:9216\n\t"
                                     "ds_read_b128 %6, %15\n\tds_read_b128 %7, %15 offset:256\n\tds_read_b128 %8, %15 offset:512\n\t"
                                     "ds_read_b128 %9, %15 offset:768\n\tds_read_b128 %10, %15 offset:1024\n\tds_read_b128 %11, %15 offset:1280\n\t"
                                     "ds_read_b128 %12, %15 offset:1536\n\tds_read_b128 %13, %15 offset:1792\n\ts_waitcnt lgkmcnt(0)"
                                     : "=&v"(a[0][0]), "=&v"(a[1][0]), "=&v"(a[0][1]), "=&v"(a[1][1]), "=&v"(a[0][2]), "=&v"(a[1][2]),
                                       "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]),
                                       "=&v"(x[6]), "=&v"(x[7])
                                     : "v"(addr), "v"(xaddr) : "memory");
        // (two features at a time: a lone column block would multiply three times in a row into one accumulator)
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            u32x4 b[2];                                       // word q of x[i] holds features 2q (low half) and 2q+1 (high half) of token i
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int pp = 0; pp < 4; ++pp) b[h][pp] = __builtin_amdgcn_perm(x[2 * pp + 1][j >> 1], x[2 * pp][j >> 1], h ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb)
                        acc[nb][j + h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[nb][pl]), __builtin_bit_cast(bf16x8, b[h]),
                                                                                 acc[nb][j + h], 0, 0, 0);
        }
    };
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
        for (int j = 0; j < 8; ++j) tot[nb][j] = floatx4{-0.f, -0.f, -0.f, -0.f};      // (plus the first share: that share)
    if (ts < te) {
        int64_t ahead = ts;                                   // the step to be requested next
        int wa = 0, set = 0;
        issue(0, ahead);
        next(ahead, wa);
        issue(1, ahead);
        next(ahead, wa);
        for (int w = 0; w < 4 && ts + w * XTT_STEP < te; ++w) {
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[nb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int64_t tb = ts + w * XTT_STEP; tb < te; tb += 4 * XTT_STEP) {
                wait_vmcnt<LOADS + XLOADS>();                      // this wave's loads of the step have landed
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_barrier();                 // everybody's have, and the stage of the step before is free
                __builtin_amdgcn_sched_barrier(0);
                issue(set == 0 ? 2 : set - 1, ahead);
                next(ahead, wa);
                multiply(set);
                set = set == 2 ? 0 : set + 1;
            }
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) tot[nb][j][e] += acc[nb][j][e];
        }
        wait_vmcnt<0>();                                      // (what was fetched past the end)
    }
    // D layout: row (k within block) = 4*(lane/16) + e, col = lane%16 -> feature 8*lc + j of the panel
    if (dcol >= K) return;                                    // (d_in is a multiple of 8: a lane's features are all in or all out)
    float* dst = partial + ((int64_t)split * K + dcol) * RP + nb0 * 16 + lg * 4;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) *reinterpret_cast<floatx4*>(dst + j * RP + nb * 16) = tot[nb][j];
}

struct XttDev {
    const bf16_t* X; int64_t ldx, M, K;
    const bf16_t* TpackT; int64_t m_pad;
    float* partial; int64_t tok_per_split;
    int one;
};
template <int NB, bool ALONE, int CAP>
__global__ __launch_bounds__(ALONE ? 64 * XttAlone<NB>::WAVES : 256) __attribute__((amdgpu_waves_per_eu(ALONE ? XttAlone<NB>::WAVES / 4 : NB == 2 ? 2 : 1))) void xtt_bf16_many_kernel(const KBatch<XttDev, CAP> tb) {
    uint32_t bx, by;
    const XttDev& a = tb.a[kbatch_find(tb, bx, by)];
    if constexpr (ALONE) xtt_alone_body<NB>(a.X, a.ldx, a.M, a.K, a.TpackT, a.m_pad, a.partial, a.tok_per_split, bx, by);
    else xtt_bf16_body<NB>(a.X, a.ldx, a.M, a.K, a.TpackT, a.m_pad, a.partial, a.tok_per_split, a.one, bx, by);
}

// Products of several layers that read the same activations (q, k and v; gate and up), up to four with up to 16 columns each: X is read once
// for all of them.  The form above with the column blocks of NB products; products of the same launch with an X of their own (NB = 1) take it too.  Eight
// waves: four panels by two halves of the column blocks (NB = 1: the second half only loads).  Sums and bits are those of a product by itself
struct XttGroupDev {
    const bf16_t* X; int64_t ldx, M, K, m_pad, tok_per_split;
    int nb, one;
    const bf16_t* T[kXShare]; float* partial[kXShare];
};
template <int NB>
struct XttGroup {
    static constexpr int NBW = NB <= 2 ? 1 : 2, WAVES = 8;
    static constexpr int LOADS = (3 * NB + WAVES - 1) / WAVES, XLOADS = 32 / WAVES;
    static constexpr int STAGE = (LOADS * WAVES + 32) * 1024;
};
template <int NB>
__device__ __forceinline__ void xtt_group_body(const XttGroupDev& a, uint32_t bx, uint32_t by) {
    typedef XttGroup<NB> S;
    constexpr int SEGS = 3 * NB, NBW = S::NBW, WAVES = S::WAVES, LOADS = S::LOADS, XLOADS = S::XLOADS, STAGE = S::STAGE, X_AT = LOADS * WAVES * 1024;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) char xtt_smem[];          // [3 stages]: [segments][16 rows][32 tokens], [4 panels][32 tokens][128 features]
    typedef __attribute__((address_space(3))) void* lptr_t;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = lane & 15, lg = lane >> 4, panel = wave & 3, half = wave >> 2;
    const int64_t M = a.M, K = a.K, m_pad = a.m_pad, ldx = a.ldx;
    const int split = (int)by;
    const int64_t ts = (int64_t)split * a.tok_per_split, te = min(ts + a.tok_per_split, m_pad);
    const int64_t dcol = ((int64_t)bx * 4 + panel) * XTT_PANEL + lc * 8;
    const bf16_t* xcol = a.X + min(dcol, K - 8);              // (features past the end repeat the last, unstored)
    // segment pl NB + nb: plane pl of product nb (past the last: that once more, into rows nobody reads)
    const bf16_t* tsrc[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int seg = min(wave + WAVES * i, SEGS - 1);
        tsrc[i] = a.T[seg % NB] + (int64_t)(16 * (seg / NB) + (lane >> 2)) * m_pad + (lane & 3) * 8;
    }
    auto next = [&](int64_t& tb, int& w) __attribute__((always_inline)) {      // (the shares are every fourth step, one share after the other)
        tb += 4 * XTT_STEP;
        if (tb >= te) tb = ++w < 4 ? ts + w * XTT_STEP : te;
    };
    auto issue = [&](int set, int64_t tb) __attribute__((always_inline)) {
        tb = min(tb, te - XTT_STEP);                          // (past the last step: that once more)
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(tsrc[i] + tb), (lptr_t)(xtt_smem + set * STAGE + (wave + WAVES * i) * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < XLOADS; ++i) {                    // (rows past M meet zero planes)
            const int q = half * XLOADS + i;
            __builtin_amdgcn_global_load_lds((gptr_t)(xcol + min(tb + 4 * q + lg, M - 1) * ldx), (lptr_t)(xtt_smem + set * STAGE + X_AT + panel * 8192 + q * 1024), 16, 0, 0);
        }
    };
    // this wave's column blocks nb0, nb0 + 1 (of three the last one twice)
    const int nb0 = half * NBW, nb1 = min(nb0 + 1, NB - 1);
    floatx4 acc[NBW][8], tot[NBW][8];
    auto multiply = [&](int set) __attribute__((always_inline)) {
        u32x4 t[NBW][3], x[8];
        const uint32_t at = (uint32_t)(uintptr_t)(lptr_t)(xtt_smem + set * STAGE + lc * 64 + lg * 16), addr0 = at + nb0 * 1024, addr1 = at + nb1 * 1024;
        const uint32_t xaddr = (uint32_t)(uintptr_t)(lptr_t)(xtt_smem + set * STAGE + X_AT + panel * 8192 + lg * 2048 + lc * 16);
        if constexpr (NBW == 1)
            asm volatile("ds_read_b128 %0, %11\n\tds_read_b128 %1, %11 offset:%13\n\tds_read_b128 %2, %11 offset:%14\n\t"
                                     "ds_read_b128 %3, %12\n\tds_read_b128 %4, %12 offset:256\n\tds_read_b128 %5, %12 offset:512\n\t"
                                     "ds_read_b128 %6, %12 offset:768\n\tds_read_b128 %7, %12 offset:1024\n\tds_read_b128 %8, %12 offset:1280\n\t"
                                     "ds_read_b128 %9, %12 offset:1536\n\tds_read_b128 %10, %12 offset:1792\n\ts_waitcnt lgkmcnt(0)"
                                     : "=&v"(t[0][0]), "=&v"(t[0][1]), "=&v"(t[0][2]), "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]),
                                       "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
                                     : "v"(addr0), "v"(xaddr), "n"(NB * 1024), "n"(2 * NB * 1024) : "memory");
        else
            asm volatile("ds_read_b128 %0, %14\n\tds_read_b128 %1, %15\n\tds_read_b128 %2, %14 offset:%17\n\t"
                                     "ds_read_b128 %3, %15 offset:%17\n\tds_read_b128 %4, %14 offset:%18\n\tds_read_b128 %5, %15 offset:%18\n\t"
                                     "ds_read_b128 %6, %16\n\tds_read_b128 %7, %16 offset:256\n\tds_read_b128 %8, %16 offset:512\n\t"
                                     "ds_read_b128 %9, %16 offset:768\n\tds_read_b128 %10, %16 offset:1024\n\tds_read_b128 %11, %16 offset:1280\n\t"
                                     "ds_read_b128 %12, %16 offset:1536\n\tds_read_b128 %13, %16 offset:1792\n\ts_waitcnt lgkmcnt(0)"
                                     : "=&v"(t[0][0]), "=&v"(t[NBW - 1][0]), "=&v"(t[0][1]), "=&v"(t[NBW - 1][1]), "=&v"(t[0][2]), "=&v"(t[NBW - 1][2]),
                                       "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]),
                                       "=&v"(x[6]), "=&v"(x[7])
                                     : "v"(addr0), "v"(addr1), "v"(xaddr), "n"(NB * 1024), "n"(2 * NB * 1024) : "memory");
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            u32x4 b[2];                                       // word q of x[i] holds features 2q (low half) and 2q+1 (high half) of token i
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int pp = 0; pp < 4; ++pp) b[h][pp] = __builtin_amdgcn_perm(x[2 * pp + 1][j >> 1], x[2 * pp][j >> 1], h ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int nb = 0; nb < NBW; ++nb)
                        acc[nb][j + h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, t[nb][pl]), __builtin_bit_cast(bf16x8, b[h]),
                                                                                 acc[nb][j + h], 0, 0, 0);
        }
    };
    const bool multiplies = NB > 1 || half == 0;
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
        for (int j = 0; j < 8; ++j) tot[nb][j] = floatx4{-0.f, -0.f, -0.f, -0.f};      // (plus the first share: that share)
    if (ts < te) {
        int64_t ahead = ts;                                   // the step to be requested next
        int wa = 0, set = 0;
        issue(0, ahead);
        next(ahead, wa);
        issue(1, ahead);
        next(ahead, wa);
        for (int w = 0; w < 4 && ts + w * XTT_STEP < te; ++w) {
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[nb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int64_t tb = ts + w * XTT_STEP; tb < te; tb += 4 * XTT_STEP) {
                wait_vmcnt<LOADS + XLOADS>();                      // this wave's loads of the step have landed
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_barrier();                 // everybody's have, and the stage of the step before is free
                __builtin_amdgcn_sched_barrier(0);
                issue(set == 0 ? 2 : set - 1, ahead);
                next(ahead, wa);
                if (multiplies) multiply(set);
                set = set == 2 ? 0 : set + 1;
            }
#pragma unroll
            for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                for (int j = 0; j < 8; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) tot[nb][j][e] += acc[nb][j][e];
        }
        wait_vmcnt<0>();                                      // (what was fetched past the end)
    }
    // D layout: row (k within block) = 4*(lane/16) + e, col = lane%16 -> feature 8*lc + j of the panel
    if (dcol >= K || !multiplies) return;                     // (d_in is a multiple of 8: a lane's features are all in or all out)
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
        if (nb0 + nb >= NB) break;
        if (a.one) {                                          // the first column alone
            float* dst = a.partial[nb0 + nb] + (int64_t)split * K + dcol;
            if (lg == 0)
#pragma unroll
                for (int j = 0; j < 8; j += 4) *reinterpret_cast<floatx4*>(dst + j) = floatx4{tot[nb][j][0], tot[nb][j + 1][0], tot[nb][j + 2][0], tot[nb][j + 3][0]};
            continue;
        }
        float* dst = a.partial[nb0 + nb] + ((int64_t)split * K + dcol) * 16 + lg * 4;
#pragma unroll
        for (int j = 0; j < 8; ++j) *reinterpret_cast<floatx4*>(dst + j * 16) = tot[nb][j];
    }
}
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void xtt_group_kernel(const KBatch<XttGroupDev> tb) {
    uint32_t bx, by;
    const XttGroupDev& a = tb.a[kbatch_find(tb, bx, by)];
    switch (a.nb) {
        case 1: xtt_group_body<1>(a, bx, by); break;
        case 2: xtt_group_body<2>(a, bx, by); break;
        case 3: xtt_group_body<3>(a, bx, by); break;
        default: xtt_group_body<4>(a, bx, by); break;
    }
}

static int64_t xtt_tokens_per_split(int64_t m_pad, int nsplit) {
    const int64_t t = (m_pad + nsplit - 1) / nsplit;
    return (t + 4 * XTT_STEP - 1) / (4 * XTT_STEP) * (4 * XTT_STEP);
}

// ALONE or not, from the workgroups that the other form would have work for and their steps: where they fill the chip less than
// once, a quarter of them leaves it idle (r = 32, 16384 tokens of a 4096-wide layer, 256 workgroups of 64 steps: 58 us against 34), and
// beyond that two column blocks, which the other form has two waves a SIMD for, need short ranges or many workgroups (r = 32, 4096 tokens
// of a 9728-wide layer, 304 workgroups of 32 steps: 34 us against 28; 16384 tokens, 608 of 64: 68 against 85).  Over 72 shapes of r = 32, 48
// and 64 with more than 256 workgroups 0.58 to 1.03 of the other form's time
static bool xtt_alone(int rp, int64_t workgroups, int64_t steps) {
    return workgroups > 256 && (rp > 32 || workgroups >= 512 || steps <= 8 * workgroups);
}
template <int NB, bool ALONE, int CAP>
static hipError_t launch_xtt_nb(const KBatch<XttDev, CAP>& tb, unsigned blocks, hipStream_t st) {
    const int smem = ALONE ? 3 * XttAlone<NB>::STAGE : XTT_PANEL * NB * 16 * (int)sizeof(float);
    static bool set = false;
    if (ALONE && !set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(xtt_bf16_many_kernel<NB, ALONE, CAP>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL((xtt_bf16_many_kernel<NB, ALONE, CAP>), dim3(blocks), dim3(ALONE ? 64 * XttAlone<NB>::WAVES : 256), smem, st, tb);
    return hipGetLastError();
}
template <int CAP>
static hipError_t launch_xtt_cap(const KBatch<XttDev, CAP>& tb, unsigned blocks, int rp, bool alone, hipStream_t st) {
    switch (rp / 16) {
        case 1: return launch_xtt_nb<1, false>(tb, blocks, st);
        case 2: return alone ? launch_xtt_nb<2, true>(tb, blocks, st) : launch_xtt_nb<2, false>(tb, blocks, st);
        case 3: return alone ? launch_xtt_nb<3, true>(tb, blocks, st) : launch_xtt_nb<3, false>(tb, blocks, st);
        case 4: return alone ? launch_xtt_nb<4, true>(tb, blocks, st) : launch_xtt_nb<4, false>(tb, blocks, st);
        default: return hipErrorInvalidValue;
    }
}

// the same for a launch of up to 16 columns with products that share X: *done = false where there are none
static hipError_t launch_xtt_groups(const XttArgs* a, int n, hipStream_t st, bool* done) {
    *done = false;
    KBatch<XttGroupDev> tb;
    tb.n = 0;
    int nsplit[kBatchMax], most = 1;
    for (int m = 0; m < n; ++m) {
        if (a[m].M == 0 || a[m].K == 0) continue;
        if (a[m].rp != 16) return hipSuccess;
        int g = 0;
        for (; g < tb.n; ++g)
            if (tb.a[g].nb < kXShare && tb.a[g].X == a[m].X && tb.a[g].ldx == a[m].ldx && tb.a[g].M == a[m].M && tb.a[g].K == a[m].K && tb.a[g].m_pad == a[m].m_pad &&
                nsplit[g] == a[m].nsplit && (tb.a[g].one != 0) == a[m].one) break;
        XttGroupDev& d = tb.a[g];
        if (g == tb.n) {
            d.X = a[m].X; d.ldx = a[m].ldx; d.M = a[m].M; d.K = a[m].K; d.m_pad = a[m].m_pad;
            d.tok_per_split = xtt_tokens_per_split(a[m].m_pad, a[m].nsplit);
            d.nb = 0;
            d.one = a[m].one ? 1 : 0;
            nsplit[tb.n++] = a[m].nsplit;
        }
        d.T[d.nb] = a[m].TpackT;
        d.partial[d.nb++] = a[m].partial;
        most = d.nb > most ? d.nb : most;
    }
    if (most == 1) return hipSuccess;
    // the longest ranges first, and of equal ones those with the most columns
    KBatch<XttGroupDev> sorted;
    sorted.n = 0;
    uint64_t blocks = 0;
    bool taken[kBatchMax] = {};
    for (int i = 0; i < tb.n; ++i) {
        int at = -1;
        for (int g = 0; g < tb.n; ++g)
            if (!taken[g] && (at < 0 || tb.a[g].tok_per_split > tb.a[at].tok_per_split || (tb.a[g].tok_per_split == tb.a[at].tok_per_split && tb.a[g].nb > tb.a[at].nb))) at = g;
        taken[at] = true;
        const uint32_t gx = (uint32_t)((tb.a[at].K + 4 * XTT_PANEL - 1) / (4 * XTT_PANEL));
        sorted.first[i] = (uint32_t)blocks; sorted.gx[i] = gx; sorted.a[i] = tb.a[at];
        sorted.n++;
        blocks += (uint64_t)gx * (uint32_t)nsplit[at];
    }
    if (blocks < XTT_GROUP_MIN) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    static bool set = false;
    if (!set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(xtt_group_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 3 * XttGroup<4>::STAGE);
        if (e != hipSuccess) return e;
        set = true;
    }
    const int smem = 3 * (most <= 2 ? XttGroup<2>::STAGE : XttGroup<4>::STAGE);
    hipLaunchKernelGGL(xtt_group_kernel, dim3((unsigned)blocks), dim3(512), smem, st, sorted);
    *done = true;
    return hipGetLastError();
}

hipError_t launch_xtt_bf16_many(const XttArgs* a, int n, bool half_cu, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    if (!half_cu) {
        bool done;
        const hipError_t e = launch_xtt_groups(a, n, st, &done);
        if (e != hipSuccess || done) return e;
    }
    KBatch<XttDev> tb;
    tb.n = 0;
    int64_t busy = 0, steps = 0;
    int rp = 0;
    for (int m = 0; m < n; ++m) {
        if (a[m].M == 0 || a[m].K == 0) continue;
        if (rp == 0) rp = a[m].rp;
        if (a[m].rp != rp || a[m].nsplit < 1 || (a[m].one && rp != 16)) return hipErrorInvalidValue;
        // (ranges that hold tokens, and their steps)
        const int64_t panels = (a[m].K + XTT_PANEL - 1) / XTT_PANEL, tok = xtt_tokens_per_split(a[m].m_pad, a[m].nsplit);
        busy += panels * ((a[m].m_pad + tok - 1) / tok);
        steps += panels * (a[m].m_pad / XTT_STEP);
    }
    const bool alone = rp > 16 && xtt_alone(rp, busy, steps);
    const int panel = (alone ? 4 : 1) * XTT_PANEL;
    // the longest ranges first, so that the launch does not end on a few of them.  Up to 16 columns that pays from some 1100 workgroups on:
    // where they start more or less together, the long ones next to each other are the slower order (bases of two to ten layers, K = 2, with
    // ranges that differ, against the caller's order: below 1100 workgroups 0.97 to 1.06 of its time, 1.006 in the mean, above 0.96 to 1.03, 0.99)
    const bool sorted = rp > 16 || busy >= 1100;
    int order[kBatchMax], count = 0;
    for (int m = 0; m < n; ++m) {
        if (a[m].M == 0 || a[m].K == 0) continue;
        int at = count++;
        const int64_t tok = xtt_tokens_per_split(a[m].m_pad, a[m].nsplit);
        for (; sorted && at > 0 && xtt_tokens_per_split(a[order[at - 1]].m_pad, a[order[at - 1]].nsplit) < tok; --at) order[at] = order[at - 1];
        order[at] = m;
    }
    uint64_t blocks = 0;
    for (int i = 0; i < count; ++i) {
        const int m = order[i];
        XttDev d;
        d.X = a[m].X; d.ldx = a[m].ldx; d.M = a[m].M; d.K = a[m].K; d.TpackT = a[m].TpackT; d.m_pad = a[m].m_pad;
        d.partial = a[m].partial; d.tok_per_split = xtt_tokens_per_split(a[m].m_pad, a[m].nsplit);
        d.one = a[m].one ? 1 : 0;
        const uint32_t gx = (uint32_t)((a[m].K + panel - 1) / panel);
        tb.first[tb.n] = (uint32_t)blocks; tb.gx[tb.n] = gx; tb.a[tb.n++] = d;
        blocks += (uint64_t)gx * (uint32_t)a[m].nsplit;
    }
    if (tb.n == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    return tb.n == 1 ? launch_xtt_cap(kbatch_one(tb), (unsigned)blocks, rp, alone, st) : launch_xtt_cap(tb, (unsigned)blocks, rp, alone, st);
}

hipError_t launch_xtt_bf16(const bf16_t* X, int64_t ldx, int64_t M, int64_t K, const bf16_t* TpackT, int64_t m_pad,
                           int rp, float* partial, int nsplit, hipStream_t st) {
    const XttArgs a{X, ldx, M, K, TpackT, m_pad, rp, partial, nsplit};
    return launch_xtt_bf16_many(&a, 1, false, st);
}

// S[d][k] = sum over splits (fp64, fixed order) of partial[s][d][rp].  (One load after the other 64 of 256 rows took 17 us, 128 31)
__global__ __launch_bounds__(256) void reduce_splits_kernel(const float* __restrict__ partial, int nsplit, int64_t d,
                                                            int rp, int r, float* __restrict__ S) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= d * rp) return;
    const int k = (int)(idx % rp);
    const int64_t row = idx / rp;
    if (k >= r) return;
    double s = 0.0;
    for (int sp0 = 0; sp0 < nsplit; sp0 += 16) {            // sixteen loads in flight (past the last: that once more, left out)
        float x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = partial[(int64_t)min(sp0 + u, nsplit - 1) * d * rp + idx];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (sp0 + u < nsplit) s += (double)x[u];
    }
    S[row * r + k] = (float)s;
}

hipError_t launch_reduce_splits(const float* partial, int nsplit, int64_t d, int rp, int r, float* S, hipStream_t st) {
    if (d == 0) return hipSuccess;
    dim3 grid((unsigned)((d * rp + 255) / 256));
    hipLaunchKernelGGL(reduce_splits_kernel, grid, dim3(256), 0, st, partial, nsplit, d, rp, r, S);
    return hipGetLastError();
}

// fp32 [d][r] -> bf16 planes [3][rp][d] (hi, mid, lo); columns >= r are zero
__global__ __launch_bounds__(256) void pack_planes_kernel(const float* __restrict__ Q, int64_t d, int r, int rp,
                                                          bf16_t* __restrict__ pack) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= d * rp) return;
    const int64_t row = idx % d;
    const int k = (int)(idx / d);
    const float f = (k < r) ? Q[row * r + k] : 0.f;
    bf16_t hi, mid, lo;
    split3_bf16(f, hi, mid, lo);
    pack[((int64_t)0 * rp + k) * d + row] = hi;
    pack[((int64_t)1 * rp + k) * d + row] = mid;
    pack[((int64_t)2 * rp + k) * d + row] = lo;
}

hipError_t launch_pack_planes(const float* Q, int64_t d, int r, int rp, bf16_t* pack, hipStream_t st) {
    if (d == 0) return hipSuccess;
    dim3 grid((unsigned)((d * rp + 255) / 256));
    hipLaunchKernelGGL(pack_planes_kernel, grid, dim3(256), 0, st, Q, d, r, rp, pack);
    return hipGetLastError();
}

}  // namespace agzo
