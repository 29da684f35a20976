// fp32-storage path: every product accumulates in fp64 on the matrix cores (v_mfma_f64_16x16x4_f64) and is rounded once.
//   forward : Y = X W^T (+ eps (X B) G^T, Eq. 7 factored), optional Y store, squared-error loss from the fp64 accumulators
//   xq      : T = X Q      (tokens x r)
//   xtt     : S = X^T T    (d_in x r), T = Omega or X Q
// All three take several problems per launch (the layers of a set; both signs of a perturbed evaluation).
//
// Operand layout of the instruction: lane l supplies element (l % 16, k = l / 16) of A (rows) and of B (columns), and
// register i of the result is row 4 i + l / 16, column l % 16.  A product does not care about the order of its k, so a
// lane fetches four consecutive k of its row at once (16 bytes) and feeds them to four instructions: instruction s takes
// k = 4 (l / 16) + s of a 16-wide chunk from both operands.
#include "agzo_internal.h"

namespace agzo {

typedef double doublex4 __attribute__((ext_vector_type(4)));
template <int V> struct IC { static constexpr int value = V; };

// ---------------------------------------------------------------------------
// Forward.  64 x 64 tile per workgroup, four waves of 32 x 32, d_in in slices of 32 double buffered in LDS (32 KiB per
// workgroup, up to four workgroups per compute unit), the next slice in flight in registers.
// Bound by the fp64 rate (78.6 TFLOP/s, the same on the matrix cores and the vector units): one instruction takes 64 cycles
// for two operand registers, so that a slice is 2048 cycles of matrix work per wave against eight LDS reads and 32
// conversions.  Vector instructions take turns with it, some four cycles each (the matrix unit was busy 83 % of the time at 50 vector
// instructions a slice), so addresses are constants and 32-bit offsets from uniform bases: 34 a slice, the three forwards of
// the 0.6B-sized set on 1000 tokens 1622 and 1580 us.  (Half of the conversions, with the slices in fp64 in LDS, were lost again to twice the
// LDS reads and barriers: 1668.)  The vector-unit version it replaces (a 4 x 4 register tile per thread) converted eight values from LDS for
// every 16 multiplications, loaded without a prefetch, and ran at 7 TFLOP/s.  The small tile is for few tokens: 1000 x 1024
// outputs give one wave to each of the 1024 SIMDs.
// Launches of fewer than F32_SMALL_LAUNCH such tiles take 32 x 32 ones, four waves of 16 x 16, with four slices in flight, for layers
// of fewer than F32_SMALL: the work of a tile is a quarter, and what bounds it is no longer the matrix rate of a few compute units but the
// latency of its loads (512 tokens, 256 x 256: 32 workgroups and 17.6 us a forward, 128 and 7.6 us).  Where the large tiles fill the chip
// once and a half they are the faster ones (steps of K = 0, us with the small, the large tiles: eight layers of 64 tiles 607 and 570, sixteen
// of 32 704 and 673, two of 120 320 and 308; below, three of 64 121 and 138, seven 0.6B-sized ones on 128 tokens 376 and 463).
// Where rows are no 16-byte vectors, value-by-value loads are four times the instructions and the small tile has twice as many for its
// work: there it is launches of fewer than F32_SMALL_SCALAR (four layers of 64 tiles, 2047 wide: 478 and 386; two of 126, 198 wide: 131 and
// 120; below, one of 64 189 and 243)
// ---------------------------------------------------------------------------
constexpr int F32_SMALL = 128, F32_SMALL_LAUNCH = 400, F32_SMALL_SCALAR = 192;      // in 64 x 64 tiles
constexpr int FK = 32;      // slice of d_in: a tile row is 128 bytes in LDS
static int64_t f32_tiles(int64_t M, int64_t N) { return ((M + 63) / 64) * ((N + 63) / 64); }
// loss partials of a layer: one for every 32 x 32 or every 64 x 64 outputs, by its shape alone, so that a layer's losses have the same bits
// in every launch
static int f32_part(int64_t M, int64_t N) { return f32_tiles(M, N) < F32_SMALL ? 32 : 64; }

struct F32FwdDev {
    F32FwdArgs a;
    int tiles_m, tiles_n;
    bool fine;               // 64 x 64 tiles, but a partial for every 32 x 32 outputs, with the bits of the 32 x 32 tile
};

// byte offset of 16-byte chunk c of tile row `row` (the XOR spreads the rows of one read over the banks)
__device__ __forceinline__ int f32_lds_off(int row, int c) { return row * 128 + ((c ^ ((row >> 1) & 7)) << 4); }

// (at least two waves per SIMD: the accumulators then stay in ordinary registers; with the whole file to itself the compiler moves
// all of them to the accumulation half and back around every slice)
template <bool VEC, int FT, int CAP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void forward_f32_kernel(const KBatch<F32FwdDev, CAP> tb) {
    constexpr int FB = FT / 32, AHEAD = FT == 64 ? 1 : 4;    // 16 x 16 blocks of a wave in either direction; slices in flight
    __shared__ __align__(16) char smem[2 * 2 * FT * FK * 4];
    __shared__ double red[4];
    uint32_t bx, by;
    const F32FwdDev& d = tb.a[kbatch_find(tb, bx, by)];
    const F32FwdArgs& a = d.a;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lc = lane & 15, lg = lane >> 4;
    const int wt = (wave & 1) * 16 * FB, wo = (wave >> 1) * 16 * FB;               // the wave's tokens and outputs
    // each XCD (workgroup id mod 8) takes a contiguous run of tiles, in bands of eight token tiles per output tile
    const int count = d.tiles_m * d.tiles_n, per = count / 8;
    int lin = (int)bx;
    if (lin < per * 8) lin = (lin % 8) * per + lin / 8;
    constexpr int BAND = 8;
    const int band = lin / (BAND * d.tiles_n), first = band * BAND;
    const int rows = min(BAND, d.tiles_m - first), in_band = lin - band * BAND * d.tiles_n;
    const int tm = first + in_band % rows, tn = in_band / rows;
    const int64_t m0 = (int64_t)tm * FT, n0 = (int64_t)tn * FT;
    char* const Xs = smem;                                 // [2 buffers][FT][FK]
    char* const Ws = smem + 2 * FT * FK * 4;

    doublex4 acc[FB][FB];
#pragma unroll
    for (int i = 0; i < FB; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};

    // staging: a 16-byte chunk per thread, operand and 32 rows.  Rows past the end repeat the last one (they only feed outputs that
    // the epilogue masks), columns past d_in are zero
    const int ch = tid & 7, r0 = tid >> 3;                 // rows r0 (and r0 + 32)
    const float *xr[FB], *wr[FB];
    uint32_t xo[FB], wo_[FB];                              // (VEC: bytes from the tile's first row, a uniform base)
    const char *xb = reinterpret_cast<const char*>(a.X + m0 * a.ldx), *wb = reinterpret_cast<const char*>(a.W + n0 * a.ldw);
#pragma unroll
    for (int i = 0; i < FB; ++i) {
        const int64_t rx_ = min(m0 + r0 + 32 * i, a.M - 1), rw_ = min(n0 + r0 + 32 * i, a.N - 1);
        xr[i] = a.X + rx_ * a.ldx;
        wr[i] = a.W + rw_ * a.ldw;
        xo[i] = (uint32_t)(((rx_ - m0) * a.ldx + ch * 4) * 4);
        wo_[i] = (uint32_t)(((rw_ - n0) * a.ldw + ch * 4) * 4);
    }
    float4 rx[AHEAD][FB], rw[AHEAD][FB];
    // MASK: the slice may reach past d_in (with several slices in flight its end is loaded instead and left out: around a lane's
    // condition the compiler waits for each load before the next)
    auto load4 = [&](const float* p, int64_t k, auto MASK) __attribute__((always_inline)) -> float4 {
        constexpr bool mask = decltype(MASK)::value != 0;
        if constexpr (VEC) {
            if constexpr (!mask) return *reinterpret_cast<const float4*>(p + k);
            if constexpr (AHEAD == 1) return (k < a.K) ? *reinterpret_cast<const float4*>(p + k) : make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 v = *reinterpret_cast<const float4*>(p + min(k, a.K - 4));
            return (k < a.K) ? v : make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (AHEAD > 1 || !mask || k + e < a.K) ? p[AHEAD > 1 ? min(k + e, a.K - 1) : k + e] : 0.f;
            if constexpr (AHEAD > 1) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = k + e < a.K ? v[e] : 0.f;
            }
            return make_float4(v[0], v[1], v[2], v[3]);
        }
    };
    auto gload = [&](float4 (&x)[FB], float4 (&w)[FB], int64_t k0, auto MASK) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            x[i] = load4(xr[i], k0 + ch * 4, MASK);
            w[i] = load4(wr[i], k0 + ch * 4, MASK);
        }
    };
    auto sstore = [&](const float4 (&x)[FB], const float4 (&w)[FB], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            const int off = buf * FT * FK * 4 + f32_lds_off(r0 + 32 * i, ch);
            *reinterpret_cast<float4*>(Xs + off) = x[i];
            *reinterpret_cast<float4*>(Ws + off) = w[i];
        }
    };
    // scale: factor on the W side in fp64 (1 for the d_in slices)
    auto multiply = [&](int buf, double scale) {
#pragma unroll
        for (int c = 0; c < FK / 16; ++c) {
            float av[FB][4], bv[FB][4];
#pragma unroll
            for (int i = 0; i < FB; ++i) {
                const float4 x = *reinterpret_cast<const float4*>(Xs + buf * FT * FK * 4 + f32_lds_off(wt + i * 16 + lc, 4 * c + lg));
                const float4 w = *reinterpret_cast<const float4*>(Ws + buf * FT * FK * 4 + f32_lds_off(wo + i * 16 + lc, 4 * c + lg));
                av[i][0] = x.x; av[i][1] = x.y; av[i][2] = x.z; av[i][3] = x.w;
                bv[i][0] = w.x; bv[i][1] = w.y; bv[i][2] = w.z; bv[i][3] = w.w;
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                double ad[FB], bd[FB];
#pragma unroll
                for (int i = 0; i < FB; ++i) { ad[i] = (double)av[i][s]; bd[i] = (double)bv[i][s] * scale; }
#pragma unroll
                for (int i = 0; i < FB; ++i)
#pragma unroll
                    for (int j = 0; j < FB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ad[i], bd[j], acc[i][j], 0, 0, 0);
            }
        }
    };
    const int nfull = (int)(a.K / FK), nk = (int)((a.K + FK - 1) / FK);
    if constexpr (AHEAD == 1) {
        gload(rx[0], rw[0], 0, IC<1>{});
        sstore(rx[0], rw[0], 0);
        __syncthreads();
        int kt = 0;
        auto whole = [&](int k, auto BUF) __attribute__((always_inline)) {
            if constexpr (VEC) {
#pragma unroll
                for (int i = 0; i < FB; ++i) {
                    rx[0][i] = *reinterpret_cast<const float4*>(xb + (int64_t)k * (FK * 4) + xo[i]);
                    rw[0][i] = *reinterpret_cast<const float4*>(wb + (int64_t)k * (FK * 4) + wo_[i]);
                }
            } else {
                gload(rx[0], rw[0], (int64_t)k * FK, IC<0>{});
            }
            multiply(decltype(BUF)::value, 1.0);
            sstore(rx[0], rw[0], decltype(BUF)::value ^ 1);
            __syncthreads();
        };
        // (two slices at a time: the buffers' addresses are then constants.  Vector instructions take turns with the fp64 matrix ones)
        for (; kt + 2 < nfull; kt += 2) {
            whole(kt + 1, IC<0>{});
            whole(kt + 2, IC<1>{});
        }
        for (; kt < nk; ++kt) {                            // the last two or three slices
            if (kt + 1 < nk) gload(rx[0], rw[0], (int64_t)(kt + 1) * FK, IC<1>{});
            multiply(kt & 1, 1.0);
            if (kt + 1 < nk) sstore(rx[0], rw[0], (kt + 1) & 1);
            __syncthreads();
        }
    } else {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) gload(rx[i], rw[i], (int64_t)i * FK, IC<1>{});
        for (int k0 = 0; k0 < nk; k0 += AHEAD)
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (k0 + i >= nk) break;
                sstore(rx[i], rw[i], i & 1);
                gload(rx[i], rw[i], (int64_t)(k0 + i + AHEAD) * FK, IC<1>{});
                __syncthreads();                           // (the buffer was read two slices ago: everyone is past that)
                multiply(i & 1, 1.0);
            }
        __syncthreads();
    }
    // the rank-r term as more slices: P rows against G rows regenerated from the seed, eps applied in fp64
    auto rank_term = [&](double coef) {
        for (int k0 = 0; k0 < a.r; k0 += FK) {
            constexpr int TR = 256 / FT;                   // threads to a row of the tile
            const int row_t = tid / TR;
#pragma unroll
            for (int i = 0; i < 8 / TR; ++i) {
                const int c = (tid % TR) * (8 / TR) + i, k = k0 + 4 * c;
                float4 pv = make_float4(0.f, 0.f, 0.f, 0.f), gv = pv;
                if (k < a.r) {
                    const float* p = a.P + min(m0 + row_t, a.M - 1) * a.r;
                    pv = make_float4(p[k], p[min(k + 1, a.r - 1)], p[min(k + 2, a.r - 1)], p[min(k + 3, a.r - 1)]);
                    if (k + 1 >= a.r) pv.y = 0.f;
                    if (k + 2 >= a.r) pv.z = 0.f;
                    if (k + 3 >= a.r) pv.w = 0.f;
                    gv = philox_normal4(a.s_lo, a.s_hi, AGZO_TAG_G, (uint32_t)min(n0 + row_t, a.N - 1), (uint32_t)(k >> 2));
                    if (k + 1 >= a.r) gv.y = 0.f;
                    if (k + 2 >= a.r) gv.z = 0.f;
                    if (k + 3 >= a.r) gv.w = 0.f;
                }
                *reinterpret_cast<float4*>(Xs + f32_lds_off(row_t, c)) = pv;
                *reinterpret_cast<float4*>(Ws + f32_lds_off(row_t, c)) = gv;
            }
            __syncthreads();
            multiply(0, coef);
            __syncthreads();
        }
    };
    auto evaluate = [&](int phase) {
        double part = 0.0, quarter[FB][FB];
        auto across = [&](double v) __attribute__((always_inline)) -> double {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
            return v;
        };
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            // eight targets requested before the first is used; rows and columns past the end repeat the last (conditional on
            // uniform values only: around a lane's condition the compiler waits for each load before the next)
            float tv[FB][4];
            auto targets = [&](auto read) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < FB; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        tv[j][e] = read(min(m0 + wt + i * 16 + 4 * e + lg, a.M - 1) * a.ldt + min(n0 + wo + j * 16 + lc, a.N - 1));
            };
            if (a.target != nullptr) {
                if (a.target_dtype == AGZO_BF16) targets([&](int64_t at) { return bf16_to_f32(reinterpret_cast<const bf16_t*>(a.target)[at]); });
                else targets([&](int64_t at) { return reinterpret_cast<const float*>(a.target)[at]; });
            }
#pragma unroll
            for (int j = 0; j < FB; ++j) {
                const int64_t col = n0 + wo + j * 16 + lc;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t row = m0 + wt + i * 16 + 4 * e + lg;
                    if (row >= a.M || col >= a.N) continue;
                    const double y = acc[i][j][e];
                    if (a.Y != nullptr) a.Y[row * a.ldy + col] = (float)y;
                    if (a.target != nullptr) {
                        const double r = y - (double)tv[j][e];
                        part = fma(r, r, part);
                    }
                }
                if constexpr (FT == 64)
                    if (d.fine) {                          // as four waves of the small tile add up theirs
                        quarter[i][j] = part;
                        part = 0.0;
                    }
            }
        }
        if (a.target == nullptr) return;
        if constexpr (FT == 64)
            if (d.fine) {
#pragma unroll
                for (int off = 32; off > 0; off >>= 1)
#pragma unroll
                    for (int q = 0; q < 4; ++q) quarter[q >> 1][q & 1] += __shfl_xor(quarter[q >> 1][q & 1], off);
                const int64_t bm = (m0 + wt) / 32, bn = (n0 + wo) / 32, rows = (a.M + 31) / 32, cols = (a.N + 31) / 32;
                if (lane == 0 && bm < rows && bn < cols) a.partials[(phase * rows + bm) * cols + bn] = (quarter[0][0] + quarter[1][0]) + (quarter[0][1] + quarter[1][1]);
                return;
            }
        part = across(part);
        if (lane == 0) red[wave] = part;
        __syncthreads();
        if (tid == 0) a.partials[(int64_t)phase * count + tm * d.tiles_n + tn] = (red[0] + red[1]) + (red[2] + red[3]);
        __syncthreads();
    };
    if (a.shared) {
        // one pass over X and W for f0, f+ and f-
        evaluate(0);
        rank_term((double)a.eps_signed);
        evaluate(1);
        rank_term(-2.0 * (double)a.eps_signed);
        evaluate(2);
    } else {
        if (a.P != nullptr) rank_term((double)a.eps_signed);
        evaluate(0);
    }
}

int forward_f32_num_workgroups(int64_t M, int64_t N) {
    const int t = f32_part(M, N);
    return (int)(((M + t - 1) / t) * ((N + t - 1) / t));
}

// every row of X and W starts on 16 bytes, and the rows of a tile lie within 32 bits of its first
static bool f32_vec(const F32FwdArgs& a) {
    return a.ldx < (1 << 24) && a.ldw < (1 << 24) && a.K % 4 == 0 && a.ldx % 4 == 0 && a.ldw % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.X) | reinterpret_cast<uintptr_t>(a.W)) & 15) == 0;
}

template <int FT>
static hipError_t launch_forward_f32_tiles(const F32FwdArgs* const* a, int n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    KBatch<F32FwdDev> tb;
    tb.n = 0;
    uint64_t blocks = 0;
    bool vec = true;
    for (int i = 0; i < n; ++i) {
        F32FwdDev d;
        d.a = *a[i];
        d.tiles_m = (int)((d.a.M + FT - 1) / FT);
        d.tiles_n = (int)((d.a.N + FT - 1) / FT);
        d.fine = FT == 64 && d.a.target && f32_part(d.a.M, d.a.N) == 32;
        vec = vec && f32_vec(d.a);
        tb.first[tb.n] = (uint32_t)blocks;
        tb.gx[tb.n] = (uint32_t)((int64_t)d.tiles_m * d.tiles_n);
        blocks += tb.gx[tb.n];
        tb.a[tb.n++] = d;
    }
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(256);
    if constexpr (FT == 32)      // (the larger tile, at its limit of registers, spills more with one argument set and is 2 % slower)
        if (tb.n == 1) {
            if (vec) hipLaunchKernelGGL((forward_f32_kernel<true, FT, 1>), grid, block, 0, st, kbatch_one(tb));
            else hipLaunchKernelGGL((forward_f32_kernel<false, FT, 1>), grid, block, 0, st, kbatch_one(tb));
            return hipGetLastError();
        }
    if (vec) hipLaunchKernelGGL((forward_f32_kernel<true, FT, kBatchMax>), grid, block, 0, st, tb);
    else hipLaunchKernelGGL((forward_f32_kernel<false, FT, kBatchMax>), grid, block, 0, st, tb);
    return hipGetLastError();
}

hipError_t launch_forward_f32_many(const F32FwdArgs* a, int n, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    int order[kBatchMax], m = 0;
    for (int i = 0; i < n; ++i) {
        if (a[i].M == 0 || a[i].N == 0) continue;
        if (a[i].K < 1 || (a[i].shared && (!a[i].P || a[i].Y || !a[i].target))) return hipErrorInvalidValue;
        // deepest first, so that the launch does not end on a few long tiles
        int at = m++;
        for (; at > 0 && a[order[at - 1]].K < a[i].K; --at) order[at] = order[at - 1];
        order[at] = i;
    }
    int64_t tiles = 0;
    bool vec = true;
    for (int i = 0; i < m; ++i) {
        tiles += f32_tiles(a[order[i]].M, a[order[i]].N);
        vec = vec && f32_vec(a[order[i]]);
    }
    const F32FwdArgs *large[kBatchMax], *small[kBatchMax];
    int nl = 0, ns = 0;
    for (int i = 0; i < m; ++i) {
        const F32FwdArgs& p = a[order[i]];
        if (tiles < (vec ? F32_SMALL_LAUNCH : F32_SMALL_SCALAR) && f32_part(p.M, p.N) == 32) small[ns++] = &p;
        else large[nl++] = &p;
    }
    const hipError_t e = launch_forward_f32_tiles<64>(large, nl, st);
    return e != hipSuccess ? e : launch_forward_f32_tiles<32>(small, ns, st);
}

// Y[t][j] += eps_signed sum_k P[t][k] G[j][k] on stored outputs: the shared-forward schedule with a cross-entropy loss, which
// needs every evaluation's logits in memory.  32 tokens x 64 outputs per workgroup, fp64.
constexpr int EP_T = 32;
constexpr int EP_J = 64;

__global__ __launch_bounds__(256) void rank_term_f32_kernel(float* __restrict__ Y, int64_t ldy, int64_t M, int64_t N,
                                                            const float* __restrict__ P, int r, float eps_signed, uint32_t s_lo,
                                                            uint32_t s_hi) {
    __shared__ float Gs[EP_J][kMaxRank + 1];
    __shared__ float Ps[EP_T][kMaxRank + 1];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.y * EP_T, j0 = (int64_t)blockIdx.x * EP_J;
    const int nquad = (r + 3) / 4;
    for (int e = tid; e < EP_J * nquad; e += 256) {
        const int jj = e / nquad, q = e % nquad;
        float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        if (j0 + jj < N) z = philox_normal4(s_lo, s_hi, AGZO_TAG_G, (uint32_t)(j0 + jj), (uint32_t)q);
        const float v[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (q * 4 + i < r) Gs[jj][q * 4 + i] = v[i];
    }
    for (int e = tid; e < EP_T * r; e += 256) {
        const int tt = e / r, k = e % r;
        Ps[tt][k] = (t0 + tt < M) ? P[(t0 + tt) * r + k] : 0.f;
    }
    __syncthreads();
    const int jj = tid % EP_J;
    const int64_t j = j0 + jj;
    for (int tt = tid / EP_J; tt < EP_T; tt += 256 / EP_J) {
        const int64_t t = t0 + tt;
        if (t >= M || j >= N) continue;
        double s = 0.0;
        for (int k = 0; k < r; ++k) s = fma((double)Ps[tt][k], (double)Gs[jj][k], s);
        Y[t * ldy + j] = (float)((double)Y[t * ldy + j] + (double)eps_signed * s);
    }
}

hipError_t launch_rank_term_f32(float* Y, int64_t ldy, int64_t M, int64_t N, const float* P, int r, float eps_signed,
                                uint64_t seed, hipStream_t st) {
    if (M == 0 || N == 0) return hipSuccess;
    dim3 grid((unsigned)((N + EP_J - 1) / EP_J), (unsigned)((M + EP_T - 1) / EP_T));
    hipLaunchKernelGGL(rank_term_f32_kernel, grid, dim3(256), 0, st, Y, ldy, M, N, P, r, eps_signed, (uint32_t)seed, (uint32_t)(seed >> 32));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tall-skinny products, bound by latency at the sizes this path sees: a workgroup is 16 waves that share one block of 16
// result rows and split the contraction between them, so that the whole chip has loads in flight after one launch and no
// second one is needed to add partial sums (they meet in LDS, in wave order).  The result has up to four blocks of 16 columns.
// (The generic 64 x 64 tile kernel that these replace walked the contraction alone, with r of its 64 columns in use: 50 us at
// 512 x 256 and r = 4, now 4.6 (xq) and 5.5 (xtt); the seven layers of 1000 x 1024 .. 3072 in one launch take 22 and 17 us.)  A
// load of xq is conditional on nothing but uniform values: with conditions of a lane, and the forms for aligned and other rows
// beside each other in the loop, the compiler waited for each (34 us, and 5.0 at 512 x 256).
// ---------------------------------------------------------------------------
constexpr int SK_WAVES = 16;

struct F32SkinnyDev {
    F32SkinnyArgs a;
    int vec;
};

// the waves' 16 x 16 blocks -> sum in wave order -> out (row0 + row, col0 + col), rows < nrow, columns < r
// xq, r = 1, flag != nullptr: V is a column that is still to be divided by its norm, and the result is instead, in fp64 as the sums are.  Every workgroup
// multiplies with every value of the column, so it adds up their squares as it goes: no launch for the norm between power steps, and none that
// scales the column (4.5 us each).  A lone layer's basis, K = 3, with those launches and so, us: 64 wide on 100 tokens 30.2 and 20.9, 256 on 512 38.5 and 29.5,
// 1024 42.3 and 31.2, 4096 51.1 and 38.6, 3072 on 1000 60.0 and 47.7; a step of the 0.6B-sized layers on 1000 tokens 1665 and 1647.  One rounding less: errors against
// 64 bits 5.3 to 5.9e-8 and 4.4 to 5.1e-8
__device__ __forceinline__ double column_scale(const double* norms, int n, int* flag, bool report) {
    double sum = 0.0;
    for (int w = 0; w < n; ++w) sum += norms[w];
    if (!(sum > 0.0)) {
        if (report) *flag = 1;
        sum = 1.0;
    }
    return 1.0 / sqrt(sum);
}
template <int NB>
__device__ __forceinline__ void skinny_f32_finish(const doublex4 (&acc)[NB], double* red, int64_t row0, int64_t nrow, int r,
                                                  float* __restrict__ out, const double* norms = nullptr, int* flag = nullptr, bool first = false) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lc = lane & 15, lg = lane >> 4;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wave * 256 + (4 * e + lg) * 16 + lc] = acc[nb][e];
        __syncthreads();
        if (tid < 256) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < SK_WAVES; ++w) s += red[w * 256 + tid];
            if (flag) s *= column_scale(norms, SK_WAVES, flag, first && tid == 0);
            const int64_t row = row0 + (tid >> 4);
            const int col = nb * 16 + (tid & 15);
            if (row < nrow && col < r) out[row * r + col] = (float)s;
        }
        __syncthreads();
    }
}

// T = X Q: rows = tokens, 16-wide chunks of d_in dealt to the waves
template <int NB, bool VEC>
__device__ __forceinline__ void xq_f32_rows(const F32SkinnyArgs& a, double* red, uint32_t bx) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lc = lane & 15, lg = lane >> 4;
    const int64_t t0 = (int64_t)bx * 16;
    const float* xr = a.X + min(t0 + lc, a.M - 1) * a.ldx;
    doublex4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = doublex4{0.0, 0.0, 0.0, 0.0};
    const int nchunk = (int)((a.K + 15) / 16);
    constexpr int U = (NB == 1) ? 4 : 2;                   // chunks in flight per wave
    __shared__ double norms[NB == 1 ? SK_WAVES : 1];
    const bool norm = NB == 1 && a.flag != nullptr;        // (r = 1: the values are lane 0's of each sixteen, the others' are zero)
    double squares = 0.0;
    for (int c0 = wave; c0 < nchunk; c0 += U * SK_WAVES) {
        float x[U][4], q[U][NB][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = 16 * (int64_t)(c0 + u * SK_WAVES) + 4 * lg;
            if (c0 + u * SK_WAVES >= nchunk) break;        // (wave-uniform)
            if constexpr (VEC) {
                const float4 v = *reinterpret_cast<const float4*>(xr + min(k, a.K - 4));
                x[u][0] = v.x; x[u][1] = v.y; x[u][2] = v.z; x[u][3] = v.w;
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) x[u][s] = xr[min(k + s, a.K - 1)];
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int s = 0; s < 4; ++s) q[u][nb][s] = a.V[min(k + s, a.K - 1) * a.r + min(nb * 16 + lc, a.r - 1)];
        }
        // (never conditional on the lane: what lies past the end is read from the last place and left out)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = 16 * (int64_t)(c0 + u * SK_WAVES) + 4 * lg;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                x[u][s] = k + s < a.K ? x[u][s] : 0.f;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) q[u][nb][s] = k + s < a.K && nb * 16 + lc < a.r ? q[u][nb][s] : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c0 + u * SK_WAVES >= nchunk) break;        // (wave-uniform)
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[u][s], (double)q[u][nb][s], acc[nb], 0, 0, 0);
            if (norm)
#pragma unroll
                for (int s = 0; s < 4; ++s) squares = fma((double)q[u][0][s], (double)q[u][0][s], squares);
        }
    }
    if (norm) {
        squares += __shfl_xor(squares, 16);
        squares += __shfl_xor(squares, 32);
        if (lane == 0) norms[wave] = squares;
    }
    skinny_f32_finish<NB>(acc, red, t0, a.M, a.r, a.out, norms, NB == 1 ? a.flag : nullptr, bx == 0);
}
template <int NB>
__global__ __launch_bounds__(64 * SK_WAVES) void xq_f32_kernel(const KBatch<F32SkinnyDev> tb) {
    __shared__ double red[SK_WAVES * 256];
    uint32_t bx, by;
    const F32SkinnyDev& d = tb.a[kbatch_find(tb, bx, by)];
    if (d.vec)      // (once, around everything: where two forms of a load meet, the compiler waits for it)
        xq_f32_rows<NB, true>(d.a, red, bx);
    else
        xq_f32_rows<NB, false>(d.a, red, bx);
}

// T = X Q for one to four columns, of which the form above uses as many lanes in sixteen to load Q: a workgroup is four tokens, its four
// waves share d_in in chunks of 256, a lane multiplies four consecutive values of each token with the rows of Q that belong to them, on
// the vector units (whose fp64 rate is that of the matrix cores and far from what bounds this: the bytes of X and their latency; two
// chunks in flight).  Seven layers of 1000 x 1024 .. 3072 at r = 1: 22 us a launch above, 11 here (18 with both forms of the load of X inside
// the loop).  Shorter rows leave waves without a chunk and loads for nothing: a step on 512 tokens at r = 1 / 4, above and here, 80 / 102 and
// 86 / 114 us 256-wide, 92 / 124 and 94 / 134 512-wide, 116 / 149 and 103 / 148 1024-wide, 161 / 196 and 134 / 180 2048-wide
constexpr int XQN_TOK = 4, XQN_MIN = 1024;
template <int R, bool VEC>
__device__ __forceinline__ void xq_f32_narrow_rows(const F32SkinnyArgs& a, double (*red)[XQN_TOK * R], uint32_t bx) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t0 = (int64_t)bx * XQN_TOK, K = a.K;
    const float* xr[XQN_TOK];
#pragma unroll
    for (int t = 0; t < XQN_TOK; ++t) xr[t] = a.X + min(t0 + t, a.M - 1) * a.ldx;
    __shared__ double norms[4];
    double acc[XQN_TOK][R] = {}, squares = 0.0;
    const int64_t nchunk = (K + 255) / 256;
    constexpr int U = 2;
    for (int64_t c0 = wave; c0 < nchunk; c0 += 4 * U) {
        // (never conditional on the lane: what lies past the end is read from the last place and left out)
        float x[U][XQN_TOK][4], q[U][4][R];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = 256 * (c0 + 4 * u) + 4 * lane;
            if constexpr (VEC) {
                const int64_t kc = min(k, K - 4);
#pragma unroll
                for (int t = 0; t < XQN_TOK; ++t) {
                    const float4 v = *reinterpret_cast<const float4*>(xr[t] + kc);
                    x[u][t][0] = v.x; x[u][t][1] = v.y; x[u][t][2] = v.z; x[u][t][3] = v.w;
                }
            } else {
#pragma unroll
                for (int t = 0; t < XQN_TOK; ++t)
#pragma unroll
                    for (int s = 0; s < 4; ++s) x[u][t][s] = xr[t][min(k + s, K - 1)];
            }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < R; ++j) q[u][s][j] = a.V[min(k + s, K - 1) * R + j];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = 256 * (c0 + 4 * u) + 4 * lane;
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const double qd = (double)q[u][s][j];
                    if (R == 1) squares = fma(k + s < K ? qd : 0.0, qd, squares);
#pragma unroll
                    for (int t = 0; t < XQN_TOK; ++t) acc[t][j] = fma(k + s < K ? (double)x[u][t][s] : 0.0, k + s < K ? qd : 0.0, acc[t][j]);
                }
        }
    }
#pragma unroll
    for (int t = 0; t < XQN_TOK; ++t)
#pragma unroll
        for (int j = 0; j < R; ++j) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc[t][j] += __shfl_xor(acc[t][j], off);
            if (lane == 0) red[wave][t * R + j] = acc[t][j];
        }
    if (R == 1 && a.flag) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) squares += __shfl_xor(squares, off);
        if (lane == 0) norms[wave] = squares;
    }
    __syncthreads();
    const int e = threadIdx.x;
    if (e < XQN_TOK * R && t0 + e / R < a.M) {
        double v = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
        if (R == 1 && a.flag) v *= column_scale(norms, 4, a.flag, bx == 0 && e == 0);
        a.out[t0 * R + e] = (float)v;
    }
}
template <int R>
__global__ __launch_bounds__(256) void xq_f32_narrow_kernel(const KBatch<F32SkinnyDev> tb) {
    __shared__ double red[4][XQN_TOK * R];
    uint32_t bx, by;
    const F32SkinnyDev& d = tb.a[kbatch_find(tb, bx, by)];
    if (d.vec)
        xq_f32_narrow_rows<R, true>(d.a, red, bx);
    else
        xq_f32_narrow_rows<R, false>(d.a, red, bx);
}

// S = X^T T: rows = features, groups of four tokens dealt to the waves
template <int NB>
__global__ __launch_bounds__(64 * SK_WAVES) void xtt_f32_kernel(const KBatch<F32SkinnyDev> tb) {
    __shared__ double red[SK_WAVES * 256];
    uint32_t bx, by;
    const F32SkinnyDev& d = tb.a[kbatch_find(tb, bx, by)];
    const F32SkinnyArgs& a = d.a;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lc = lane & 15, lg = lane >> 4;
    const int64_t f0 = (int64_t)bx * 16;
    const float* xc = a.X + min(f0 + lc, a.K - 1);
    doublex4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = doublex4{0.0, 0.0, 0.0, 0.0};
    const int ngroup = (int)((a.M + 3) / 4);
    constexpr int U = (NB <= 2) ? 8 : 4;                   // groups in flight per wave
    for (int g0 = wave; g0 < ngroup; g0 += U * SK_WAVES) {
        float x[U], v[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t t = 4 * (int64_t)(g0 + u * SK_WAVES) + lg;
            // (conditional on uniform values only: around a lane's condition the compiler waits for each load before the next)
            if (g0 + u * SK_WAVES >= ngroup) break;
            const int64_t tc = min(t, a.M - 1);
            x[u] = xc[tc * a.ldx];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) v[u][nb] = a.V[tc * a.r + min(nb * 16 + lc, a.r - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = 4 * (int64_t)(g0 + u * SK_WAVES) + lg < a.M;
            x[u] = in ? x[u] : 0.f;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) v[u][nb] = in && nb * 16 + lc < a.r ? v[u][nb] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g0 + u * SK_WAVES >= ngroup) break;        // (wave-uniform)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[u], (double)v[u][nb], acc[nb], 0, 0, 0);
        }
    }
    skinny_f32_finish<NB>(acc, red, f0, a.K, a.r, a.out);
}

static bool skinny_f32_vec(const F32SkinnyArgs& a) { return a.K % 4 == 0 && a.ldx % 4 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0; }

static hipError_t launch_xq_f32_narrow(const F32SkinnyArgs* a, const int* idx, int n, int r, hipStream_t st) {
    if (n == 0) return hipSuccess;
    KBatch<F32SkinnyDev> tb;
    tb.n = 0;
    uint64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        const F32SkinnyArgs& s = a[idx[i]];
        tb.first[tb.n] = (uint32_t)blocks;
        tb.gx[tb.n] = (uint32_t)((s.M + XQN_TOK - 1) / XQN_TOK);
        blocks += tb.gx[tb.n];
        tb.a[tb.n++] = F32SkinnyDev{s, skinny_f32_vec(s)};
    }
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(256);
    switch (r) {
        case 1: hipLaunchKernelGGL(xq_f32_narrow_kernel<1>, grid, block, 0, st, tb); break;
        case 2: hipLaunchKernelGGL(xq_f32_narrow_kernel<2>, grid, block, 0, st, tb); break;
        case 3: hipLaunchKernelGGL(xq_f32_narrow_kernel<3>, grid, block, 0, st, tb); break;
        default: hipLaunchKernelGGL(xq_f32_narrow_kernel<4>, grid, block, 0, st, tb); break;
    }
    return hipGetLastError();
}

static hipError_t launch_skinny_f32(const F32SkinnyArgs* a, int n, bool transposed, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    KBatch<F32SkinnyDev> tb;
    tb.n = 0;
    uint64_t blocks = 0;
    int nb = 0, narrow[4][kBatchMax], n_narrow[4] = {};
    for (int i = 0; i < n; ++i) {
        if (a[i].M == 0 || a[i].K == 0) continue;
        if (a[i].r < 1 || a[i].r > kMaxRank) return hipErrorInvalidValue;
        const int want = (a[i].r + 15) / 16;
        if (nb == 0) nb = want;
        if (nb != want || (a[i].flag && (transposed || a[i].r != 1))) return hipErrorInvalidValue;        // one padded rank per launch
        if (!transposed && a[i].r <= 4 && a[i].K >= XQN_MIN) {
            narrow[a[i].r - 1][n_narrow[a[i].r - 1]++] = i;
            continue;
        }
        F32SkinnyDev d;
        d.a = a[i];
        d.vec = skinny_f32_vec(a[i]);
        tb.first[tb.n] = (uint32_t)blocks;
        tb.gx[tb.n] = (uint32_t)(((transposed ? a[i].K : a[i].M) + 15) / 16);
        blocks += tb.gx[tb.n];
        tb.a[tb.n++] = d;
    }
    for (int r = 1; r <= 4; ++r) {
        const hipError_t e = launch_xq_f32_narrow(a, narrow[r - 1], n_narrow[r - 1], r, st);
        if (e != hipSuccess) return e;
    }
    if (tb.n == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(64 * SK_WAVES);
    switch (nb * 2 + (transposed ? 1 : 0)) {
        case 2: hipLaunchKernelGGL(xq_f32_kernel<1>, grid, block, 0, st, tb); break;
        case 3: hipLaunchKernelGGL(xtt_f32_kernel<1>, grid, block, 0, st, tb); break;
        case 4: hipLaunchKernelGGL(xq_f32_kernel<2>, grid, block, 0, st, tb); break;
        case 5: hipLaunchKernelGGL(xtt_f32_kernel<2>, grid, block, 0, st, tb); break;
        case 6: hipLaunchKernelGGL(xq_f32_kernel<3>, grid, block, 0, st, tb); break;
        case 7: hipLaunchKernelGGL(xtt_f32_kernel<3>, grid, block, 0, st, tb); break;
        case 8: hipLaunchKernelGGL(xq_f32_kernel<4>, grid, block, 0, st, tb); break;
        case 9: hipLaunchKernelGGL(xtt_f32_kernel<4>, grid, block, 0, st, tb); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_xq_f32_many(const F32SkinnyArgs* a, int n, hipStream_t st) { return launch_skinny_f32(a, n, false, st); }
hipError_t launch_xtt_f32_many(const F32SkinnyArgs* a, int n, hipStream_t st) { return launch_skinny_f32(a, n, true, st); }

}  // namespace agzo
