// Tall-skinny products of Alg. 1 on bf16 activations (HBM-bound sweeps of X):
//   xq  : T = X Q          (N x r), contraction over d_in   -> also used for the projection P = X B
//   xtt : S = X^T T        (d_in x r), contraction over tokens (T = Omega or T = X Q)
// X is bf16; the small fp32 factor (Q, B, T, Omega) enters the matrix cores as three bf16 planes
// hi + mid + lo, whose sum is the fp32 value, so the products carry fp32-level accuracy while the
// kernels stay bound by the single read of X.  v_mfma_f32_16x16x32_bf16 throughout.
#include <type_traits>

#include "agzo_internal.h"

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

// bx: token block, by / ny: this workgroup's share of d_in (ny = 1: all of it)
// ring depth: DEEP = one workgroup per CU with as many slices in flight as LDS holds; otherwise a shallower ring that
// lets two workgroups share a CU, for launches with at least two workgroups per CU (several layers at once): while one
// waits at its barrier or on its fragment reads the other multiplies
template <int NB, bool DEEP>
struct XqRing { static constexpr int STAGES = DEEP ? ((NB == 1) ? 8 : (NB == 2) ? 6 : 4) : ((NB == 1) ? 5 : (NB == 2) ? 3 : 4); };

// a slot holds the rows of a slice and, where four waves do not share their groups evenly, groups that nobody reads: every wave
// then issues the same number of loads and waits by constants (a wait chosen among a dozen cases and a branch around each load
// cost more than the slice's matrix work)
constexpr int xq_slot_bytes(int nb) { return (XQ_TOK / 8 + 6 * nb + 3) / 4 * 4096; }

template <int NB, bool DEEP>
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

    floatx4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = floatx4{0.f, 0.f, 0.f, 0.f};

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
    // partial sums in `part` for xq_finish_kernel (a single workgroup per block would walk d_in alone, bound by latency)
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
        if constexpr (NB == 1)
            asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %10 offset:2048\n\t"
                         "ds_read_b128 %4, %10 offset:4096\n\tds_read_b128 %1, %9\n\tds_read_b128 %5, %11\n\t"
                         "ds_read_b128 %6, %11 offset:2048\n\tds_read_b128 %7, %11 offset:4096\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0][0][0]), "=&v"(b[0][0][1]), "=&v"(b[0][0][2]),
                           "=&v"(b[1][0][0]), "=&v"(b[1][0][1]), "=&v"(b[1][0][2])
                         : "v"(xaddr0), "v"(xaddr1), "v"(qaddr0), "v"(qaddr1) : "memory");
        else if constexpr (NB == 2)
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
        else if constexpr (NB == 3)
            asm volatile("ds_read_b128 %0, %20\n\tds_read_b128 %2, %22\n\tds_read_b128 %3, %22 offset:2048\n\t"
                         "ds_read_b128 %4, %22 offset:4096\n\tds_read_b128 %5, %22 offset:6144\n\t"
                         "ds_read_b128 %6, %22 offset:8192\n\tds_read_b128 %7, %22 offset:10240\n\t"
                         "ds_read_b128 %8, %22 offset:12288\n\tds_read_b128 %9, %22 offset:14336\n\t"
                         "ds_read_b128 %10, %22 offset:16384\n\tds_read_b128 %1, %21\n\tds_read_b128 %11, %23\n\t"
                         "ds_read_b128 %12, %23 offset:2048\n\tds_read_b128 %13, %23 offset:4096\n\t"
                         "ds_read_b128 %14, %23 offset:6144\n\tds_read_b128 %15, %23 offset:8192\n\t"
                         "ds_read_b128 %16, %23 offset:10240\n\tds_read_b128 %17, %23 offset:12288\n\t"
                         "ds_read_b128 %18, %23 offset:14336\n\tds_read_b128 %19, %23 offset:16384\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0][0][0]), "=&v"(b[0][1][0]), "=&v"(b[0][2][0]),
                           "=&v"(b[0][0][1]), "=&v"(b[0][1][1]), "=&v"(b[0][2][1]), "=&v"(b[0][0][2]), "=&v"(b[0][1][2]),
                           "=&v"(b[0][2][2]), "=&v"(b[1][0][0]), "=&v"(b[1][1][0]), "=&v"(b[1][2][0]), "=&v"(b[1][0][1]),
                           "=&v"(b[1][1][1]), "=&v"(b[1][2][1]), "=&v"(b[1][0][2]), "=&v"(b[1][1][2]), "=&v"(b[1][2][2])
                         : "v"(xaddr0), "v"(xaddr1), "v"(qaddr0), "v"(qaddr1) : "memory");
        else
            asm volatile("ds_read_b128 %0, %26\n\tds_read_b128 %2, %28\n\tds_read_b128 %3, %28 offset:2048\n\t"
                         "ds_read_b128 %4, %28 offset:4096\n\tds_read_b128 %5, %28 offset:6144\n\t"
                         "ds_read_b128 %6, %28 offset:8192\n\tds_read_b128 %7, %28 offset:10240\n\t"
                         "ds_read_b128 %8, %28 offset:12288\n\tds_read_b128 %9, %28 offset:14336\n\t"
                         "ds_read_b128 %10, %28 offset:16384\n\tds_read_b128 %11, %28 offset:18432\n\t"
                         "ds_read_b128 %12, %28 offset:20480\n\tds_read_b128 %13, %28 offset:22528\n\tds_read_b128 %1, %27\n\t"
                         "ds_read_b128 %14, %29\n\tds_read_b128 %15, %29 offset:2048\n\tds_read_b128 %16, %29 offset:4096\n\t"
                         "ds_read_b128 %17, %29 offset:6144\n\tds_read_b128 %18, %29 offset:8192\n\t"
                         "ds_read_b128 %19, %29 offset:10240\n\tds_read_b128 %20, %29 offset:12288\n\t"
                         "ds_read_b128 %21, %29 offset:14336\n\tds_read_b128 %22, %29 offset:16384\n\t"
                         "ds_read_b128 %23, %29 offset:18432\n\tds_read_b128 %24, %29 offset:20480\n\t"
                         "ds_read_b128 %25, %29 offset:22528\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0][0][0]), "=&v"(b[0][1][0]), "=&v"(b[0][2][0]),
                           "=&v"(b[0][3][0]), "=&v"(b[0][0][1]), "=&v"(b[0][1][1]), "=&v"(b[0][2][1]), "=&v"(b[0][3][1]),
                           "=&v"(b[0][0][2]), "=&v"(b[0][1][2]), "=&v"(b[0][2][2]), "=&v"(b[0][3][2]), "=&v"(b[1][0][0]),
                           "=&v"(b[1][1][0]), "=&v"(b[1][2][0]), "=&v"(b[1][3][0]), "=&v"(b[1][0][1]), "=&v"(b[1][1][1]),
                           "=&v"(b[1][2][1]), "=&v"(b[1][3][1]), "=&v"(b[1][0][2]), "=&v"(b[1][1][2]), "=&v"(b[1][2][2]),
                           "=&v"(b[1][3][2])
                         : "v"(xaddr0), "v"(xaddr1), "v"(qaddr0), "v"(qaddr1) : "memory");
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[sub]), __builtin_bit_cast(bf16x8, b[sub][nb][pl]),
                                                                      acc[nb], 0, 0, 0);
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
    // D layout: row (token) = 4*(lane/16) + e, col (k) = lane%16
    if (part != nullptr) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t t = t0 + wave * 16 + lg * 4 + e;
                if (t < m_pad) part[((int64_t)split * m_pad + t) * RP + nb * 16 + lm] = acc[nb][e];
            }
        return;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int k = nb * 16 + lm;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t t = t0 + wave * 16 + lg * 4 + e;
            const float v = (t < M && k < r) ? acc[nb][e] : 0.f;
            if (t < M && k < r && T != nullptr) T[t * r + k] = v;
            if (t < M && Xext != nullptr) store_ext(Xext, t, k, RP, v);
            if (TpackT != nullptr && t < m_pad) {
                bf16_t hi, mid, lo;
                split3_bf16(v, hi, mid, lo);
                TpackT[((int64_t)0 * RP + k) * m_pad + t] = hi;
                TpackT[((int64_t)1 * RP + k) * m_pad + t] = mid;
                TpackT[((int64_t)2 * RP + k) * m_pad + t] = lo;
            }
        }
    }
}

// what a launch needs per product (the layers of a model)
struct XqDev {
    const bf16_t* X; int64_t ldx, M, K;
    const bf16_t* Qpack; int r;
    float* T; bf16_t* TpackT; int64_t m_pad; float* part;   // part: NULL unless ns > 1
    int ns; int64_t rows;
    bf16_t* Xext;
};
template <int NB, bool DEEP, int CAP>
__global__ __launch_bounds__(256) void xq_bf16_many_kernel(const KBatch<XqDev, CAP> tb) {
    uint32_t bx, by;
    const XqDev& a = tb.a[kbatch_find(tb, bx, by)];
    xq_bf16_body<NB, DEEP>(a.X, a.ldx, a.M, a.K, a.Qpack, a.r, a.T, a.TpackT, a.m_pad, a.part, a.Xext, bx, by, (uint32_t)a.ns);
}

// sums the d_in splits of xq in fixed order and writes what the unsplit kernel's epilogue writes; one thread per (t, k)
__device__ __forceinline__ void xq_finish_body(const float* __restrict__ part, int nsplit, int64_t rows, int64_t M,
                                               int64_t m_pad, int r, int rp, float* __restrict__ T,
                                               bf16_t* __restrict__ TpackT, bf16_t* __restrict__ Xext, uint32_t bx) {
    const int64_t idx = (int64_t)bx * 256 + threadIdx.x;
    if (idx >= rows * rp) return;
    const int64_t t = idx / rp;
    const int k = (int)(idx - t * rp);
    // (eight splits' loads in flight; conditional on uniform values only - around a lane's condition the compiler waits for each
    // load before the next - and what lies behind the last token or column is left out below)
    float v = 0.f;
    const float* src = part + (t < m_pad ? t : m_pad - 1) * rp + k;
    for (int s0 = 0; s0 < nsplit; s0 += 8) {
        float x[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) x[s] = s0 + s < nsplit ? src[(int64_t)(s0 + s) * m_pad * rp] : 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) v += x[s];
    }
    if (!(t < M && k < r)) v = 0.f;
    if (t < M && k < r && T != nullptr) T[t * r + k] = v;
    if (t < M && Xext != nullptr) store_ext(Xext, t, k, rp, v);
    if (TpackT != nullptr && t < m_pad) {
        bf16_t hi, mid, lo;
        split3_bf16(v, hi, mid, lo);
        TpackT[((int64_t)0 * rp + k) * m_pad + t] = hi;
        TpackT[((int64_t)1 * rp + k) * m_pad + t] = mid;
        TpackT[((int64_t)2 * rp + k) * m_pad + t] = lo;
    }
}

template <int CAP>
__global__ __launch_bounds__(256) void xq_finish_many_kernel(const KBatch<XqDev, CAP> tb, int rp) {
    uint32_t bx, by;
    const XqDev& a = tb.a[kbatch_find(tb, bx, by)];
    xq_finish_body(a.part, a.ns, a.rows, a.M, a.m_pad, a.r, rp, a.T, a.TpackT, a.Xext, bx);
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

template <int NB, bool DEEP, int CAP>
static hipError_t launch_xq_many_ring(const KBatch<XqDev, CAP>& tb, unsigned blocks, hipStream_t st) {
    const int smem = XqRing<NB, DEEP>::STAGES * xq_slot_bytes(NB);
    static bool set = false;
    if (!set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(xq_bf16_many_kernel<NB, DEEP, CAP>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, smem);
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL((xq_bf16_many_kernel<NB, DEEP, CAP>), dim3(blocks), dim3(256), smem, st, tb);
    return hipGetLastError();
}
template <int NB, int CAP>
static hipError_t launch_xq_many_nb(const KBatch<XqDev, CAP>& tb, unsigned blocks, hipStream_t st) {
    // (the result does not depend on the ring's depth: same slices, same order)
    if (NB <= 2 && blocks >= 512) return launch_xq_many_ring<NB, false>(tb, blocks, st);
    return launch_xq_many_ring<NB, true>(tb, blocks, st);
}

template <int CAP>
static hipError_t launch_xq_cap(const KBatch<XqDev, CAP>& tb, unsigned blocks, int rp, hipStream_t st) {
    switch (rp / 16) {
        case 1: return launch_xq_many_nb<1>(tb, blocks, st);
        case 2: return launch_xq_many_nb<2>(tb, blocks, st);
        case 3: return launch_xq_many_nb<3>(tb, blocks, st);
        case 4: return launch_xq_many_nb<4>(tb, blocks, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_xq_bf16_many(const XqArgs* a, int n, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    KBatch<XqDev> tb, fin;
    tb.n = fin.n = 0;
    uint64_t blocks = 0, fin_blocks = 0;
    int rp = 0;
    for (int m = 0; m < n; ++m) {
        if (a[m].M == 0) continue;
        if (rp == 0) rp = a[m].rp;
        if (a[m].rp != rp) return hipErrorInvalidValue;       // one padded rank per launch
        XqDev d;
        d.X = a[m].X; d.ldx = a[m].ldx; d.M = a[m].M; d.K = a[m].K; d.Qpack = a[m].Qpack; d.r = a[m].r;
        d.T = a[m].T; d.TpackT = a[m].TpackT; d.m_pad = a[m].m_pad;
        d.rows = a[m].TpackT ? a[m].m_pad : a[m].M;
        d.Xext = a[m].Xext;
        d.ns = a[m].part ? xq_splits(a[m].m_pad, a[m].K) : 1;
        d.part = d.ns > 1 ? a[m].part : nullptr;
        const uint32_t gx = (uint32_t)((d.rows + XQ_TOK - 1) / XQ_TOK);
        tb.first[tb.n] = (uint32_t)blocks; tb.gx[tb.n] = gx; tb.a[tb.n++] = d;
        blocks += (uint64_t)gx * (uint32_t)d.ns;
        if (d.ns > 1) {
            const uint32_t fx = (uint32_t)((d.rows * rp + 255) / 256);
            fin.first[fin.n] = (uint32_t)fin_blocks; fin.gx[fin.n] = fx; fin.a[fin.n++] = d;
            fin_blocks += fx;
        }
    }
    if (tb.n == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull || fin_blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipError_t e = tb.n == 1 ? launch_xq_cap(kbatch_one(tb), (unsigned)blocks, rp, st) : launch_xq_cap(tb, (unsigned)blocks, rp, st);
    if (e != hipSuccess || fin.n == 0) return e;
    const dim3 fin_grid((unsigned)fin_blocks);
    if (fin.n == 1) hipLaunchKernelGGL(xq_finish_many_kernel<1>, fin_grid, dim3(256), 0, st, kbatch_one(fin), rp);
    else hipLaunchKernelGGL(xq_finish_many_kernel<kBatchMax>, fin_grid, dim3(256), 0, st, fin, rp);
    return hipGetLastError();
}

hipError_t launch_xq_bf16(const bf16_t* X, int64_t ldx, int64_t M, int64_t K, const bf16_t* Qpack, int r, int rp,
                          float* T, bf16_t* TpackT, int64_t m_pad, float* part, bf16_t* Xext, hipStream_t st) {
    const XqArgs a{X, ldx, M, K, Qpack, r, rp, T, TpackT, m_pad, part, Xext};
    return launch_xq_bf16_many(&a, 1, st);
}

// ---------------------------------------------------------------------------
// xtt: workgroup = (panel of 128 features) x (token range); its four waves take 32-token steps in turn and add their sums in LDS.
// ALONE (r > 16 only): a wave has a panel of its own and takes the four waves' steps one wave after the other: the same sums in the
// same order, a quarter of the workgroups, and no adding of 128 rows of up to 64 columns in LDS, which takes longer than the few
// steps it follows.
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
template <int NB, bool ALONE>
__device__ __forceinline__ void xtt_bf16_body(const bf16_t* __restrict__ X, int64_t ldx, int64_t M, int64_t K,
                                              const bf16_t* __restrict__ TpackT, int64_t m_pad,
                                              float* __restrict__ partial, int64_t tok_per_split, uint32_t bx, uint32_t by) {
    constexpr int RP = NB * 16;
    extern __shared__ __align__(16) float sbuf[];   // [XTT_PANEL][RP]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lc = lane & 15, lg = lane >> 4;
    const int64_t db = ((int64_t)bx * (ALONE ? 4 : 1) + (ALONE ? wave : 0)) * XTT_PANEL;
    if (ALONE && db >= K) return;
    const int split = (int)by;
    const int64_t ts = (int64_t)split * tok_per_split;
    const int64_t te = min(ts + tok_per_split, m_pad);

    floatx4 acc[NB][8];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[nb][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int64_t dcol = db + lc * 8;
    const bool din = dcol < K;
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
    // A wave's steps: every fourth of the range, from its own number on; ALONE: the four waves' steps one wave after the other, and
    // their sums added in that order (tot).  Either way the same bits.  Two register sets in turn: moved from one to the other at the
    // end of a step, the loads would be waited for there
    floatx4 tot[ALONE ? NB : 1][8] = {};
    int64_t tb = ts + (ALONE ? 0 : wave * XTT_STEP);
    if (tb < te) {
        uint4 v0[8], v1[8];
        Frag a0[NB][3], a1[NB][3];
        load_step(tb, v0, a0);
        if constexpr (!ALONE) {
            for (; tb < te; tb += 2 * STRIDE) {
                load_step(min(tb + STRIDE, te - XTT_STEP), v1, a1);
                multiply(v0, a0);
                if (tb + STRIDE >= te) break;
                load_step(min(tb + 2 * STRIDE, te - XTT_STEP), v0, a0);
                multiply(v1, a1);
            }
        } else {
            int w = 0;
            bool first = true;
            // the step at tb, with the loads of the one behind it, which may be the first of the next wave's; false: there is none
            auto step = [&](uint4 (&v)[8], Frag (&a)[NB][3], uint4 (&v2)[8], Frag (&a2)[NB][3]) __attribute__((always_inline)) -> bool {
                int wn = w;
                int64_t tn = tb + STRIDE;
                if (tn >= te) tn = (++wn < 4) ? ts + wn * XTT_STEP : te;
                const bool more = tn < te;
                load_step(more ? tn : tb, v2, a2);
                multiply(v, a);
                if (wn != w || !more) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            tot[nb][j] = first ? acc[nb][j] : tot[nb][j] + acc[nb][j];
                            acc[nb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
                        }
                    first = false;
                }
                tb = tn;
                w = wn;
                return more;
            };
            while (step(v0, a0, v1, a1) && step(v1, a1, v0, a0)) {}
        }
    }
    // D layout: row (k within block) = 4*(lane/16) + e, col = lane%16 -> feature db + 8*lc + j
    if constexpr (ALONE) {
        if (!din) return;                          // (d_in is a multiple of 8: a lane's features are all in or all out)
        float* dst = partial + ((int64_t)split * K + dcol) * RP + lg * 4;
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<floatx4*>(dst + j * RP + nb * 16) = tot[nb][j];
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

struct XttDev {
    const bf16_t* X; int64_t ldx, M, K;
    const bf16_t* TpackT; int64_t m_pad;
    float* partial; int64_t tok_per_split;
};
template <int NB, bool ALONE, int CAP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NB == 2 ? 2 : 1))) void xtt_bf16_many_kernel(const KBatch<XttDev, CAP> tb) {
    uint32_t bx, by;
    const XttDev& a = tb.a[kbatch_find(tb, bx, by)];
    xtt_bf16_body<NB, ALONE>(a.X, a.ldx, a.M, a.K, a.TpackT, a.m_pad, a.partial, a.tok_per_split, bx, by);
}

static int64_t xtt_tokens_per_split(int64_t m_pad, int nsplit) {
    const int64_t t = (m_pad + nsplit - 1) / nsplit;
    return (t + 4 * XTT_STEP - 1) / (4 * XTT_STEP) * (4 * XTT_STEP);
}

// ALONE or not, from the workgroups that the other form would have work for and their steps: where they fill the chip less than
// once, a quarter of them leaves it idle (r = 32, 16384 tokens of a 4096-wide layer, 256 workgroups of 64 steps: 65 us against 33), and
// beyond that the adding is worth avoiding for short ranges (seven 4B-sized layers, 512 tokens, 832 of 4 steps: 15 us against 25 at
// r = 32, 28 against 55 at r = 64) and, where it allows one workgroup per compute unit (r > 32), for long ones too once
// there are many (4096 tokens, 1860 of some 16 steps: 129 us against 163 at r = 64, 103 against 130 at r = 48, but 78
// against 70 at r = 32; one 9728-wide layer, 304 of 32 steps: 67 against 52 at r = 64)
static bool xtt_alone(int rp, int64_t workgroups, int64_t steps) {
    return workgroups > 256 && (steps <= 8 * workgroups || (rp > 32 && workgroups >= 1024));
}
template <int NB, bool ALONE, int CAP>
static hipError_t launch_xtt_nb(const KBatch<XttDev, CAP>& tb, unsigned blocks, hipStream_t st) {
    const size_t smem = ALONE ? 0 : (size_t)XTT_PANEL * NB * 16 * sizeof(float);
    hipLaunchKernelGGL((xtt_bf16_many_kernel<NB, ALONE, CAP>), dim3(blocks), dim3(256), smem, st, tb);
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

hipError_t launch_xtt_bf16_many(const XttArgs* a, int n, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    KBatch<XttDev> tb;
    tb.n = 0;
    int64_t busy = 0, steps = 0;
    int rp = 0;
    for (int m = 0; m < n; ++m) {
        if (a[m].M == 0 || a[m].K == 0) continue;
        if (rp == 0) rp = a[m].rp;
        if (a[m].rp != rp || a[m].nsplit < 1) return hipErrorInvalidValue;
        // (ranges that hold tokens, and their steps)
        const int64_t panels = (a[m].K + XTT_PANEL - 1) / XTT_PANEL, tok = xtt_tokens_per_split(a[m].m_pad, a[m].nsplit);
        busy += panels * ((a[m].m_pad + tok - 1) / tok);
        steps += panels * (a[m].m_pad / XTT_STEP);
    }
    const bool alone = rp > 16 && xtt_alone(rp, busy, steps);
    const int panel = (alone ? 4 : 1) * XTT_PANEL;
    uint64_t blocks = 0;
    for (int m = 0; m < n; ++m) {
        if (a[m].M == 0 || a[m].K == 0) continue;
        XttDev d;
        d.X = a[m].X; d.ldx = a[m].ldx; d.M = a[m].M; d.K = a[m].K; d.TpackT = a[m].TpackT; d.m_pad = a[m].m_pad;
        d.partial = a[m].partial; d.tok_per_split = xtt_tokens_per_split(a[m].m_pad, a[m].nsplit);
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
    return launch_xtt_bf16_many(&a, 1, st);
}

// S[d][k] = sum over splits (fp64, fixed order) of partial[s][d][rp]
__global__ __launch_bounds__(256) void reduce_splits_kernel(const float* __restrict__ partial, int nsplit, int64_t d,
                                                            int rp, int r, float* __restrict__ S) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= d * rp) return;
    const int k = (int)(idx % rp);
    const int64_t row = idx / rp;
    if (k >= r) return;
    double s = 0.0;
    for (int sp = 0; sp < nsplit; ++sp) s += (double)partial[(int64_t)sp * d * rp + idx];
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
