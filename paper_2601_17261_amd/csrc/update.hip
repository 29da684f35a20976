// In-place rank-r sweep of Alg. 2 (restore / update line, Eq. 10):
//     W[i][j] -= (lr * g + shift) * sum_k G[i][k] * B[j][k]
// (shift = 0 for the update alone; shift = eps makes it the printed last line of Alg. 2, which takes the perturbation
// out and applies the update in one sweep).
// W is read and written exactly once (HBM-bound); G is regenerated from the Philox seed (the d_out x d_in
// direction Z = G B^T never exists in memory); B (d_in x r fp32) is small and stays in L2.  fp32
// accumulation, one rounding to the storage type on the store.
#include <type_traits>

#include "agzo_internal.h"

namespace agzo {

constexpr int UP_TI = 32;    // rows (d_out) per tile
constexpr int UP_TJ = 256;   // cols (d_in) per tile
constexpr int UP_TR = 4;     // rows per thread
constexpr int UP_BS = UP_TJ + 4;   // a row of the transposed B tile: 16 ranks of 4 columns in 64 banks
constexpr int UPD_MAX = 16;  // matrices of one launch

struct UpdF32Item {
    float* W;
    const float* B;
    const double* g_dev;
    int64_t ldw, d_out, d_in;
    uint32_t blk0, njb;   // first workgroup of this matrix, its tiles across
    uint32_t s_lo, s_hi;
    float lr;
    int r;
    int vec;              // rows start on 16 bytes
};
struct UpdF32Batch {
    int n;
    float shift;
    UpdF32Item it[UPD_MAX];
};

// fp32 weights keep exact fp32 products on the vector units: a workgroup takes 32 x 256 elements, a lane two runs of four
// columns in four rows.  HBM-bound, so the weights are requested before the generator and the products run (B's rows before
// them: loads return in order).  B's tile is one run of floats, read as such and turned in LDS, a row padded by 4 so that 16
// ranks of 4 columns fall on 64 banks; r is taken four at a time (the sum's order is k either way) and leaves the registers
// for the weights.  The matrices of a model share one launch (workgroups find theirs from the running block counts).
// The seven of a 1024-wide set, r = 16, 126 MB read and written, against 64 x 256 tiles that turned B through one bank, read W
// last and took a launch each: 107 -> 24 us (5.2 TB/s); a 2560-wide set 299 -> 144 (5.6 TB/s); three matrices at r = 64
// 101 -> 34 (generator and products); 1001 x 1003 and 777 x 2049, r = 7, 42 -> 13; 4096 x 12288, r = 1, 61 -> 59.  Tiles of
// 64 rows (two waves a SIMD, not four): 29, 155, 43, 13, 60; of 16 rows: 25, 158, 45, 12, 59.
// Rows that start on 16 bytes but end inside a run of four are read value by value in their last tile only.  Tiles take one form or the
// other around everything (where two forms of a load meet, the compiler waits for it): 4096 x 4094, rows of 4096, r = 1, 34.3 us with the
// earlier tiles, 36.5 value by value, 33.7 so; 31 x 70001 7.1, 11.3 and 5.9.
template <bool VEC>   // whole aligned runs of four
__device__ __forceinline__ void update_f32_tile(const UpdF32Item& u, float shift, int64_t i0, int64_t j0) {
    extern __shared__ __align__(16) float up_smem[];
    const int64_t ldw = u.ldw, d_out = u.d_out, d_in = u.d_in;
    const int r = u.r, nquad = (r + 3) / 4;
    float4* Gs = reinterpret_cast<float4*>(up_smem);        // [UP_TI][nquad]
    float* Bt = up_smem + UP_TI * nquad * 4;                // [4 nquad][UP_BS]
    const int tid = threadIdx.x;
    const int tx = tid & 31;          // columns 4 tx + 128 h of the tile
    const int ty = tid >> 5;          // rows ty + 8 s
    const int64_t jc = j0 + tx * 4;
    float* Wt = u.W + jc;
    const int64_t jl = d_in - 1, jv = jl & ~(int64_t)3;   // the last column, the last whole run of four

    // the tile's rows of B are one run of floats
    const float* Bj = u.B + j0 * r;
    const int n_b = (int)min((int64_t)UP_TJ, d_in - j0) * r;
    const int step_j = 256 / r, step_k = 256 % r;
    int bj = tid / r, bk = tid % r;
#pragma unroll 4
    for (int q = 0; q < r; ++q) {
        Bt[bk * UP_BS + bj] = Bj[min(tid + q * 256, n_b - 1)];
        bj += step_j;
        bk += step_k;
        if (bk >= r) { bk -= r; ++bj; }
    }
    for (int k = r; k < 4 * nquad; ++k) Bt[k * UP_BS + tid] = 0.f;
    // rows and columns past the end read the last ones, which are not stored
    float4 w[UP_TR][2];
#pragma unroll
    for (int s = 0; s < UP_TR; ++s) {
        const float* p = u.W + min(i0 + ty + 8 * s, d_out - 1) * ldw;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t j = jc + 128 * h;
            if constexpr (VEC)
                w[s][h] = *reinterpret_cast<const float4*>(p + min(j, jv));
            else
                w[s][h] = make_float4(p[min(j, jl)], p[min(j + 1, jl)], p[min(j + 2, jl)], p[min(j + 3, jl)]);
        }
    }

    // G tile from the seed: one Philox call = 4 columns of one row
    for (int e = tid; e < UP_TI * nquad; e += 256) {
        const int ii = e / nquad, q = e % nquad;
        float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i0 + ii < d_out) z = philox_normal4(u.s_lo, u.s_hi, AGZO_TAG_G, (uint32_t)(i0 + ii), (uint32_t)q);
        if (q * 4 + 1 >= r) z.y = 0.f;
        if (q * 4 + 2 >= r) z.z = 0.f;
        if (q * 4 + 3 >= r) z.w = 0.f;
        Gs[e] = z;
    }
    __syncthreads();

    const float coef = -fmaf(u.lr, u.g_dev ? (float)(*u.g_dev) : 1.0f, shift);
    float acc[UP_TR][8];
#pragma unroll
    for (int s = 0; s < UP_TR; ++s)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[s][c] = 0.f;
    for (int q = 0; q < nquad; ++q) {
        float b[4][8];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 v = *reinterpret_cast<const float4*>(&Bt[(q * 4 + k) * UP_BS + h * 128 + tx * 4]);
                b[k][4 * h] = v.x; b[k][4 * h + 1] = v.y; b[k][4 * h + 2] = v.z; b[k][4 * h + 3] = v.w;
            }
#pragma unroll
        for (int s = 0; s < UP_TR; ++s) {
            const float4 g4 = Gs[(ty + 8 * s) * nquad + q];
            const float g[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[s][c] = fmaf(g[k], b[k][c], acc[s][c]);
        }
    }

#pragma unroll
    for (int s = 0; s < UP_TR; ++s) {
        const int64_t i = i0 + ty + 8 * s;
        if (i >= d_out) continue;
        float* p = Wt + i * ldw;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float4 v = w[s][h];
            v.x = fmaf(coef, acc[s][4 * h], v.x);
            v.y = fmaf(coef, acc[s][4 * h + 1], v.y);
            v.z = fmaf(coef, acc[s][4 * h + 2], v.z);
            v.w = fmaf(coef, acc[s][4 * h + 3], v.w);
            const int64_t left = d_in - jc - 128 * h;
            if constexpr (VEC) {
                if (left > 0) *reinterpret_cast<float4*>(p + 128 * h) = v;
            } else {
                if (left > 0) p[128 * h] = v.x;
                if (left > 1) p[128 * h + 1] = v.y;
                if (left > 2) p[128 * h + 2] = v.z;
                if (left > 3) p[128 * h + 3] = v.w;
            }
        }
    }
}

__global__ __launch_bounds__(256) void update_f32_kernel(const UpdF32Batch tb) {
    int m = 0;
    while (m + 1 < tb.n && blockIdx.x >= tb.it[m + 1].blk0) ++m;
    const UpdF32Item& u = tb.it[m];
    const uint32_t local = blockIdx.x - u.blk0;
    const int64_t i0 = (int64_t)(local / u.njb) * UP_TI, j0 = (int64_t)(local % u.njb) * UP_TJ;
    if (u.vec && ((u.d_in & 3) == 0 || j0 + UP_TJ <= u.d_in)) update_f32_tile<true>(u, tb.shift, i0, j0);
    else update_f32_tile<false>(u, tb.shift, i0, j0);
}

// ---------------------------------------------------------------------------
// bf16 storage: the outer product G B^T runs on the matrix cores (v_mfma_f32_32x32x16_bf16,
// K = r padded to 16).  A small preparation kernel writes both factors once, already split hi + lo in
// bf16 and already in the register order the matrix instruction wants (coef = -lr g folded into G), so
// the sweep itself holds no generator and no conversions of the factors: it is a read-add-write of W.
// Products hi*hi, hi*lo, lo*hi are accumulated: relative error 2^-16 of the increment.
//
// Roles: A-operand rows = rows i of W (G), B-operand columns = columns j of W (basis rows), interleaved
// over eight instructions (column c of instruction m is j = 8 c + m), so that a lane ends up with eight
// consecutive columns of one row (16 bytes) and a half-wave with 512 contiguous bytes.
// A wave owns 32 rows x 256 columns; the four waves of a workgroup share the basis fragments in LDS.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
union FragU {
    uint4 u;
    bf16x8 v;
};

// eight fp32 values -> hi and lo bf16 fragments
__device__ __forceinline__ void split_frag(const float (&f)[8], FragU& hi, FragU& lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[i] = pack_bf16x2(f[2 * i], f[2 * i + 1]);
        const float r0 = f[2 * i] - __uint_as_float(h[i] << 16);
        const float r1 = f[2 * i + 1] - __uint_as_float(h[i] & 0xFFFF0000u);
        l[i] = pack_bf16x2(r0, r1);
    }
    hi.u = make_uint4(h[0], h[1], h[2], h[3]);
    lo.u = make_uint4(l[0], l[1], l[2], l[3]);
}

constexpr int UM_ROWS = 32;     // rows of W per wave
constexpr int UM_COLS = 256;    // columns of W per workgroup

// fragment stores (uint4 units):
//   Gf [row block ib][kc][plane][lane]        lane = (i % 32) + 32 * lh,      k = 16 kc + 8 lh + 0..7
//   Bf [col block jb][kc][plane][m][lane]     lane = c + 32 * lh, j = 256 jb + 8 c + m, same k
__device__ __forceinline__ void prep_fragment(uint4* __restrict__ Gf, uint4* __restrict__ Bf, int64_t n_g, int64_t n_b,
                                              int nk, int64_t d_out, int64_t d_in, const float* __restrict__ B, int r,
                                              uint32_t s_lo, uint32_t s_hi, float lr, float shift,
                                              const double* __restrict__ g_dev, int64_t t) {
    float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    FragU hi, lo;
    if (t < n_g) {
        const int lane = (int)(t & 63), kc = (int)((t >> 6) % nk);
        const int64_t ib = (t >> 6) / nk;
        const int64_t i = ib * UM_ROWS + (lane & 31);
        const int k0 = 16 * kc + 8 * (lane >> 5);
        if (i < d_out && k0 < r) {
            const float coef = -fmaf(lr, g_dev ? (float)(*g_dev) : 1.0f, shift);
            const float4 z0 = philox_normal4(s_lo, s_hi, AGZO_TAG_G, (uint32_t)i, (uint32_t)(k0 >> 2));
            f[0] = z0.x; f[1] = z0.y; f[2] = z0.z; f[3] = z0.w;
            if (k0 + 4 < r) {
                const float4 z1 = philox_normal4(s_lo, s_hi, AGZO_TAG_G, (uint32_t)i, (uint32_t)((k0 >> 2) + 1));
                f[4] = z1.x; f[5] = z1.y; f[6] = z1.z; f[7] = z1.w;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) f[q] = (k0 + q < r) ? coef * f[q] : 0.f;
        }
        split_frag(f, hi, lo);
        uint4* dst = Gf + ((ib * nk + kc) * 2) * 64 + lane;
        dst[0] = hi.u;
        dst[64] = lo.u;
    } else if (t < n_g + n_b) {
        const int64_t u = t - n_g;
        const int lane = (int)(u & 63), m = (int)((u >> 6) & 7), kc = (int)((u >> 9) % nk);
        const int64_t jb = (u >> 9) / nk;
        const int64_t j = jb * UM_COLS + 8 * (lane & 31) + m;
        const int k0 = 16 * kc + 8 * (lane >> 5);
        if (j < d_in) {
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (k0 + q < r) f[q] = B[j * r + k0 + q];
        }
        split_frag(f, hi, lo);
        uint4* dst = Bf + (((jb * nk + kc) * 2) * 8 + m) * 64 + lane;
        dst[0] = hi.u;
        dst[8 * 64] = lo.u;
    }
}

__global__ __launch_bounds__(256) void update_prep_kernel(uint4* __restrict__ Gf, uint4* __restrict__ Bf,
                                                          int64_t n_g, int64_t n_b, int nk, int64_t d_out,
                                                          int64_t d_in, const float* __restrict__ B, int r,
                                                          uint32_t s_lo, uint32_t s_hi, float lr, float shift,
                                                          const double* __restrict__ g_dev) {
    prep_fragment(Gf, Bf, n_g, n_b, nk, d_out, d_in, B, r, s_lo, s_hi, lr, shift, g_dev, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// Several matrices in one pair of launches (Alg. 2 updates every layer once the scalar g is known): the table is a
// kernel argument, a workgroup finds its matrix from the running block counts (uniform, a handful of scalar compares).
struct UpdItem {
    bf16_t* W;
    uint4 *Gf, *Bf;
    const float* B;
    const double* g_dev;
    int64_t ldw, d_out, d_in, n_g, n_b;
    uint32_t prep_blk0, sweep_blk0;   // first workgroup of this matrix in the two launches
    uint32_t s_lo, s_hi;
    float lr;
    int r, njb, row_iters;
};
struct UpdBatch {
    int n;
    UpdItem it[UPD_MAX];
};

__global__ __launch_bounds__(256) void update_prep_many_kernel(const UpdBatch tb, int nk) {
    int m = 0;
    while (m + 1 < tb.n && blockIdx.x >= tb.it[m + 1].prep_blk0) ++m;
    const UpdItem& u = tb.it[m];
    prep_fragment(u.Gf, u.Bf, u.n_g, u.n_b, nk, u.d_out, u.d_in, u.B, u.r, u.s_lo, u.s_hi, u.lr, 0.f, u.g_dev,
                  (int64_t)(blockIdx.x - u.prep_blk0) * 256 + threadIdx.x);
}

template <int NK>   // NK = rp / 16
__device__ __forceinline__ void sweep_columns(bf16_t* __restrict__ W, int64_t ldw, int64_t d_out, int64_t d_in,
                                              const uint4* __restrict__ Gf, const uint4* __restrict__ Bf, int row_iters,
                                              int64_t jb, int64_t by) {
    extern __shared__ __align__(16) uint4 um_smem[];   // [NK][2][8][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, lh = lane >> 5;
    {
        const uint4* src = Bf + jb * (NK * 2 * 8 * 64);
#pragma unroll
        for (int e = 0; e < NK * 4; ++e) um_smem[e * 256 + tid] = src[e * 256 + tid];
    }
    __syncthreads();
    const int64_t jc = jb * UM_COLS + 8 * c;     // this lane's eight consecutive columns
    const bool col_ok = jc < d_in;               // d_in is a multiple of 8: the piece is all in or all out
    const uint32_t voff = (uint32_t)((4 * lh * ldw + 8 * c) * 2);   // bytes from the tile's corner; ldw < 2^28 (host check)

    for (int it = 0; it < row_iters; ++it) {
        const int64_t ib = (by * row_iters + it) * 4 + wave;
        const int64_t i0 = ib * UM_ROWS;
        if (i0 >= d_out) break;                  // wave-uniform
        // this lane's rows: i0 + 8 (e / 4) + 4 lh + e % 4.  Addresses = a wave-uniform row base (scalar registers) plus
        // one 32-bit lane offset, instead of sixteen 64-bit pointers per lane
        char* tile;
        {   // kept in scalar registers: passing the halves through readfirstlane stops the compiler from turning the
            // sixteen row addresses into per-lane 64-bit induction variables of the row loop
            const uint64_t a = reinterpret_cast<uint64_t>(W + i0 * ldw + jb * UM_COLS);
            const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
            tile = reinterpret_cast<char*>(((uint64_t)hi << 32) | lo);
        }
        uint4 wv[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t i = i0 + 8 * (e >> 2) + 4 * lh + (e & 3);
            wv[e] = make_uint4(0, 0, 0, 0);
            if (col_ok && i < d_out)
                wv[e] = *reinterpret_cast<const uint4*>(tile + (int64_t)(8 * (e >> 2) + (e & 3)) * ldw * 2 + voff);
        }
        floatx16 z[8];
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) z[m][e] = 0.f;
#pragma unroll
        for (int kc = 0; kc < NK; ++kc) {
            FragU gh, gl;
            gh.u = Gf[((ib * NK + kc) * 2) * 64 + lane];
            gl.u = Gf[((ib * NK + kc) * 2 + 1) * 64 + lane];
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                FragU bh, bl;
                bh.u = um_smem[((kc * 2) * 8 + m) * 64 + lane];
                bl.u = um_smem[((kc * 2 + 1) * 8 + m) * 64 + lane];
                z[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gh.v, bh.v, z[m], 0, 0, 0);
                z[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gh.v, bl.v, z[m], 0, 0, 0);
                z[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gl.v, bh.v, z[m], 0, 0, 0);
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t i = i0 + 8 * (e >> 2) + 4 * lh + (e & 3);
            if (!(col_ok && i < d_out)) continue;
            uint32_t* pw = reinterpret_cast<uint32_t*>(&wv[e]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float w0 = __uint_as_float(pw[q] << 16), w1 = __uint_as_float(pw[q] & 0xFFFF0000u);
                pw[q] = pack_bf16x2(w0 + z[2 * q][e], w1 + z[2 * q + 1][e]);
            }
            *reinterpret_cast<uint4*>(tile + (int64_t)(8 * (e >> 2) + (e & 3)) * ldw * 2 + voff) = wv[e];
        }
    }
}

template <int NK>
__global__ __launch_bounds__(256, 2) void update_mfma_kernel(bf16_t* __restrict__ W, int64_t ldw, int64_t d_out,
                                                             int64_t d_in, const uint4* __restrict__ Gf,
                                                             const uint4* __restrict__ Bf, int row_iters) {
    sweep_columns<NK>(W, ldw, d_out, d_in, Gf, Bf, row_iters, blockIdx.x, blockIdx.y);
}

template <int NK>
__global__ __launch_bounds__(256, 2) void update_mfma_many_kernel(const UpdBatch tb) {
    int m = 0;
    while (m + 1 < tb.n && blockIdx.x >= tb.it[m + 1].sweep_blk0) ++m;
    const UpdItem& u = tb.it[m];
    const uint32_t local = blockIdx.x - u.sweep_blk0, by = local / (uint32_t)u.njb;
    sweep_columns<NK>(u.W, u.ldw, u.d_out, u.d_in, u.Gf, u.Bf, u.row_iters, local - by * (uint32_t)u.njb, by);
}

// ---------------------------------------------------------------------------
// bf16 storage, r = 1 (the paper's operating point): the perturbation is an outer product g b^T of two vectors, so the
// sweep is one read-multiply-add-write of W on the vector units with nothing prepared beforehand: a wave owns 16 rows
// x 512 columns, lane l < 16 regenerates the Gaussian value of row l once and the wave passes it around; a lane keeps
// its eight basis values in registers and has all 16 row pieces in flight before the first store.  Exact fp32
// products, one rounding to bf16.
// ---------------------------------------------------------------------------
constexpr int U1_ROWS = 16;     // rows per wave
constexpr int U1_COLS = 512;    // columns per wave (8 per lane)

__device__ __forceinline__ void update_rank1_bf16_body(bf16_t* __restrict__ W, int64_t ldw, int64_t d_out, int64_t d_in,
                                                       const float* __restrict__ B, uint32_t s_lo, uint32_t s_hi, float lr,
                                                       float shift, const double* __restrict__ g_dev, uint32_t bx, uint32_t by) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t i0 = ((int64_t)by * 4 + wave) * U1_ROWS;
    const int64_t jc = (int64_t)bx * U1_COLS + 8 * lane;
    if (i0 >= d_out) return;                               // wave-uniform
    const float coef = -fmaf(lr, g_dev ? (float)(*g_dev) : 1.0f, shift);
    float gmine = 0.f;
    if (lane < U1_ROWS && i0 + lane < d_out) gmine = coef * philox_normal4(s_lo, s_hi, AGZO_TAG_G, (uint32_t)(i0 + lane), 0u).x;
    const bool col_ok = jc < d_in;                          // d_in is a multiple of 8: the piece is all in or all out
    float b[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) b[c] = col_ok ? B[jc + c] : 0.f;
    uint4 wv[U1_ROWS];
#pragma unroll
    for (int e = 0; e < U1_ROWS; ++e) {
        wv[e] = make_uint4(0, 0, 0, 0);
        if (col_ok && i0 + e < d_out) wv[e] = *reinterpret_cast<const uint4*>(W + (i0 + e) * ldw + jc);
    }
#pragma unroll
    for (int e = 0; e < U1_ROWS; ++e) {
        const float g = __shfl(gmine, e);
        if (!(col_ok && i0 + e < d_out)) continue;
        uint32_t* pw = reinterpret_cast<uint32_t*>(&wv[e]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float w0 = __uint_as_float(pw[q] << 16), w1 = __uint_as_float(pw[q] & 0xFFFF0000u);
            pw[q] = pack_bf16x2(w0 + g * b[2 * q], w1 + g * b[2 * q + 1]);
        }
        *reinterpret_cast<uint4*>(W + (i0 + e) * ldw + jc) = wv[e];
    }
}

__global__ __launch_bounds__(256) void update_rank1_bf16_kernel(bf16_t* __restrict__ W, int64_t ldw, int64_t d_out, int64_t d_in,
                                                                const float* __restrict__ B, uint32_t s_lo, uint32_t s_hi,
                                                                float lr, float shift, const double* __restrict__ g_dev) {
    update_rank1_bf16_body(W, ldw, d_out, d_in, B, s_lo, s_hi, lr, shift, g_dev, blockIdx.x, blockIdx.y);
}

struct U1Dev {
    bf16_t* W; int64_t ldw, d_out, d_in;
    const float* B; const double* g_dev;
    uint32_t s_lo, s_hi; float lr;
};
__global__ __launch_bounds__(256) void update_rank1_bf16_many_kernel(const KBatch<U1Dev> tb) {
    uint32_t bx, by;
    const U1Dev& a = tb.a[kbatch_find(tb, bx, by)];
    update_rank1_bf16_body(a.W, a.ldw, a.d_out, a.d_in, a.B, a.s_lo, a.s_hi, a.lr, 0.f, a.g_dev, bx, by);
}

size_t update_workspace_bytes(int dtype, int64_t d_out, int64_t d_in, int r) {
    if (dtype != AGZO_BF16) return 0;
    const int64_t nk = (r + 15) / 16;
    const int64_t nib = (d_out + UM_ROWS - 1) / UM_ROWS, njb = (d_in + UM_COLS - 1) / UM_COLS;
    return (size_t)(nib * nk * 2 * 64 + njb * nk * 2 * 8 * 64) * sizeof(uint4);
}

// more rows per workgroup (fewer reloads of the basis fragments) once the grid still covers the chip a few times
static int sweep_row_iters(int64_t njb, int64_t ngroups) {
    int row_iters = 1;
    while (row_iters < 4 && njb * (ngroups / (2 * row_iters)) >= 2048) row_iters *= 2;
    return row_iters;
}

template <int NK>
static hipError_t launch_mfma(bf16_t* W, int64_t ldw, int64_t d_out, int64_t d_in, const uint4* Gf, const uint4* Bf,
                              hipStream_t st) {
    const int64_t njb = (d_in + UM_COLS - 1) / UM_COLS;
    const int64_t ngroups = (d_out + 4 * UM_ROWS - 1) / (4 * UM_ROWS);
    const int row_iters = sweep_row_iters(njb, ngroups);
    dim3 grid((unsigned)njb, (unsigned)((ngroups + row_iters - 1) / row_iters));
    const size_t smem = (size_t)NK * 2 * 8 * 64 * sizeof(uint4);
    hipLaunchKernelGGL((update_mfma_kernel<NK>), grid, dim3(256), smem, st, W, ldw, d_out, d_in, Gf, Bf, row_iters);
    return hipGetLastError();
}

hipError_t launch_update_f32_many(const UpdateDesc* d, int n, hipStream_t st, float shift) {
    if (n < 1 || n > UPD_MAX) return hipErrorInvalidValue;
    UpdF32Batch tb;
    tb.n = 0;
    tb.shift = shift;
    int64_t blocks = 0;
    int rp = 0;
    for (int m = 0; m < n; ++m) {
        if (d[m].d_out == 0 || d[m].d_in == 0) continue;
        const bool vec = (d[m].ldw & 3) == 0 && (reinterpret_cast<uintptr_t>(d[m].W) & 15) == 0;
        const int64_t njb = (d[m].d_in + UP_TJ - 1) / UP_TJ;
        tb.it[tb.n++] = UpdF32Item{static_cast<float*>(d[m].W), d[m].B, d[m].g_dev, d[m].ldw, d[m].d_out, d[m].d_in,
                                   (uint32_t)blocks, (uint32_t)njb, (uint32_t)d[m].seed, (uint32_t)(d[m].seed >> 32),
                                   d[m].lr, d[m].r, vec ? 1 : 0};
        blocks += njb * ((d[m].d_out + UP_TI - 1) / UP_TI);
        rp = max(rp, (d[m].r + 3) / 4 * 4);
    }
    if (tb.n == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    const size_t smem = (size_t)(UP_TI + UP_BS) * rp * sizeof(float);
    static bool set = false;
    if (!set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(update_f32_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (UP_TI + UP_BS) * kMaxRank * (int)sizeof(float));
        if (e != hipSuccess) return e;
        set = true;
    }
    hipLaunchKernelGGL(update_f32_kernel, dim3((unsigned)blocks), dim3(256), smem, st, tb);
    return hipGetLastError();
}

hipError_t launch_update(void* W, int dtype, int64_t ldw, int64_t d_out, int64_t d_in, const float* B, int r,
                         uint64_t seed, float lr, const double* g_dev, void* workspace, hipStream_t st, float shift) {
    if (d_out == 0 || d_in == 0) return hipSuccess;
    // fp32 storage keeps exact fp32 products (VALU); bf16 storage takes the matrix-core outer product
    if (dtype != AGZO_BF16) {
        const UpdateDesc d{W, B, g_dev, ldw, d_out, d_in, seed, lr, r};
        return launch_update_f32_many(&d, 1, st, shift);
    }
    if (r == 1) {
        const dim3 grid((unsigned)((d_in + U1_COLS - 1) / U1_COLS), (unsigned)((d_out + 4 * U1_ROWS - 1) / (4 * U1_ROWS)));
        hipLaunchKernelGGL(update_rank1_bf16_kernel, grid, dim3(256), 0, st, static_cast<bf16_t*>(W), ldw, d_out, d_in, B,
                           (uint32_t)seed, (uint32_t)(seed >> 32), lr, shift, g_dev);
        return hipGetLastError();
    }
    if (!workspace || ldw >= (1LL << 28)) return hipErrorInvalidValue;   // the sweep's lane offsets are 32-bit
    const int nk = (r + 15) / 16;
    const int64_t nib = (d_out + UM_ROWS - 1) / UM_ROWS, njb = (d_in + UM_COLS - 1) / UM_COLS;
    const int64_t n_g = nib * nk * 64, n_b = njb * nk * 8 * 64;
    uint4* Gf = static_cast<uint4*>(workspace);
    uint4* Bf = Gf + nib * nk * 2 * 64;
    hipLaunchKernelGGL(update_prep_kernel, dim3((unsigned)((n_g + n_b + 255) / 256)), dim3(256), 0, st, Gf, Bf, n_g, n_b,
                       nk, d_out, d_in, B, r, (uint32_t)seed, (uint32_t)(seed >> 32), lr, shift, g_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    bf16_t* Wb = static_cast<bf16_t*>(W);
    switch (nk) {
        case 1: return launch_mfma<1>(Wb, ldw, d_out, d_in, Gf, Bf, st);
        case 2: return launch_mfma<2>(Wb, ldw, d_out, d_in, Gf, Bf, st);
        case 3: return launch_mfma<3>(Wb, ldw, d_out, d_in, Gf, Bf, st);
        default: return launch_mfma<4>(Wb, ldw, d_out, d_in, Gf, Bf, st);
    }
}

// bf16 matrices of one padded rank (nk = ceil(r / 16) the same for all), at most UPD_MAX of them: one preparation
// launch and one sweep for the lot.  The workspace holds the fragments of all of them back to back.
// bf16 matrices with r = 1, at most kBatchMax: one launch of the rank-1 sweep for all of them (no scratch)
hipError_t launch_update_rank1_many(const UpdateDesc* d, int n, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    KBatch<U1Dev> tb;
    tb.n = 0;
    uint64_t blocks = 0;
    for (int m = 0; m < n; ++m) {
        if (d[m].d_out == 0 || d[m].d_in == 0) continue;
        if (d[m].r != 1) return hipErrorInvalidValue;
        const uint32_t gx = (uint32_t)((d[m].d_in + U1_COLS - 1) / U1_COLS);
        const uint64_t gy = (uint64_t)((d[m].d_out + 4 * U1_ROWS - 1) / (4 * U1_ROWS));
        tb.first[tb.n] = (uint32_t)blocks; tb.gx[tb.n] = gx;
        tb.a[tb.n++] = U1Dev{static_cast<bf16_t*>(d[m].W), d[m].ldw, d[m].d_out, d[m].d_in, d[m].B, d[m].g_dev,
                             (uint32_t)d[m].seed, (uint32_t)(d[m].seed >> 32), d[m].lr};
        blocks += gx * gy;
    }
    if (tb.n == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(update_rank1_bf16_many_kernel, dim3((unsigned)blocks), dim3(256), 0, st, tb);
    return hipGetLastError();
}

hipError_t launch_update_many(const UpdateDesc* d, int n, int nk, void* workspace, hipStream_t st) {
    if (n < 1 || n > UPD_MAX || !workspace) return hipErrorInvalidValue;
    UpdBatch tb;
    tb.n = 0;
    uint4* ws = static_cast<uint4*>(workspace);
    int64_t prep_blocks = 0, sweep_blocks = 0;
    for (int m = 0; m < n; ++m) {
        if (d[m].d_out == 0 || d[m].d_in == 0) continue;
        if (d[m].ldw >= (1LL << 28)) return hipErrorInvalidValue;
        UpdItem& u = tb.it[tb.n++];
        const int64_t nib = (d[m].d_out + UM_ROWS - 1) / UM_ROWS, njb = (d[m].d_in + UM_COLS - 1) / UM_COLS;
        const int64_t ngroups = (d[m].d_out + 4 * UM_ROWS - 1) / (4 * UM_ROWS);
        u.W = static_cast<bf16_t*>(d[m].W);
        u.Gf = ws;
        u.Bf = ws + nib * nk * 2 * 64;
        ws = u.Bf + njb * nk * 2 * 8 * 64;
        u.B = d[m].B;
        u.g_dev = d[m].g_dev;
        u.ldw = d[m].ldw; u.d_out = d[m].d_out; u.d_in = d[m].d_in;
        u.n_g = nib * nk * 64; u.n_b = njb * nk * 8 * 64;
        u.s_lo = (uint32_t)d[m].seed; u.s_hi = (uint32_t)(d[m].seed >> 32);
        u.lr = d[m].lr; u.r = d[m].r;
        u.njb = (int)njb;
        u.row_iters = sweep_row_iters(njb, ngroups);
        u.prep_blk0 = (uint32_t)prep_blocks;
        u.sweep_blk0 = (uint32_t)sweep_blocks;
        prep_blocks += (u.n_g + u.n_b + 255) / 256;
        sweep_blocks += njb * ((ngroups + u.row_iters - 1) / u.row_iters);
    }
    if (tb.n == 0) return hipSuccess;
    if (prep_blocks > 0x7FFFFFFFLL || sweep_blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(update_prep_many_kernel, dim3((unsigned)prep_blocks), dim3(256), 0, st, tb, nk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t smem = (size_t)nk * 2 * 8 * 64 * sizeof(uint4);
    const dim3 grid((unsigned)sweep_blocks);
    switch (nk) {
        case 1: hipLaunchKernelGGL((update_mfma_many_kernel<1>), grid, dim3(256), smem, st, tb); break;
        case 2: hipLaunchKernelGGL((update_mfma_many_kernel<2>), grid, dim3(256), smem, st, tb); break;
        case 3: hipLaunchKernelGGL((update_mfma_many_kernel<3>), grid, dim3(256), smem, st, tb); break;
        case 4: hipLaunchKernelGGL((update_mfma_many_kernel<4>), grid, dim3(256), smem, st, tb); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int update_many_max() { return UPD_MAX; }

// Dense Gaussian sweep (Eq. 7, the branch for parameters that are not linear-layer weights; Alg. 2 perturb / restore /
// update lines): theta[i][j] += coef * z(i, j), z from Philox stream AGZO_TAG_DENSE, coef = scale * (*g_dev or 1).
// A thread takes the same four columns of DENSE_ROWS rows, a Philox call each, with what it reads requested before the first.  The
// generator bounds this kernel, not the 4 - 8 bytes per value it moves.  (A 64-bit division a thread for its place, one row a thread
// and the two halves of every Philox product by themselves: the estimator over seven 0.6B-sized layers 419 us a step, 408 so.)  Rows
// that four columns do not divide are read and written value by value, each load in its place: there half the threads hide less of that
// latency than they save of the generator's (fp32, 982 x 1183: 5.1 us with a row a thread, 6.2 with two; 1024 x 2047 6.8 and 7.2; 8192 x
// 4095 62 and 62), except in large bf16 blocks (8192 x 4095: 49 and 47); all with a generator of 59 instructions a value.  With 50 a
// value 8192 x 4096 in bf16 takes 39.0 us instead of 43.9
template <typename T, bool VEC, int DENSE_ROWS>
__global__ __launch_bounds__(256) void dense_axpy_kernel(T* __restrict__ theta, int64_t rows, int64_t cols, int64_t ld,
                                                         int64_t nquad, int64_t items, uint32_t s_lo, uint32_t s_hi, float scale,
                                                         const double* __restrict__ g_dev) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= items) return;
    int64_t group, quad;
    if (items <= 0xFFFFFFFFLL) {
        const uint32_t q = (uint32_t)idx / (uint32_t)nquad;
        group = q;
        quad = (uint32_t)idx - q * (uint32_t)nquad;
    } else {
        group = idx / nquad;
        quad = idx - group * nquad;
    }
    const int64_t row = group * DENSE_ROWS;
    const int n = (int)min((int64_t)DENSE_ROWS, rows - row);
    T* p = theta + row * ld + quad * 4;
    typedef typename std::conditional<sizeof(T) == 4, float4, uint2>::type vec_t;
    vec_t v[DENSE_ROWS];
    if constexpr (VEC) {
#pragma unroll
        for (int i = 0; i < DENSE_ROWS; ++i) v[i] = *reinterpret_cast<const vec_t*>(p + min(i, n - 1) * ld);
    }
    const float coef = g_dev ? (float)((double)scale * *g_dev) : scale;
#pragma unroll
    for (int i = 0; i < DENSE_ROWS; ++i) {
        if (i >= n) break;
        const float4 z4 = philox_normal4(s_lo, s_hi, AGZO_TAG_DENSE, (uint32_t)(row + i), (uint32_t)quad);
        const float z[4] = {z4.x, z4.y, z4.z, z4.w};
        T* pi = p + i * ld;
        if constexpr (VEC) {
            if constexpr (sizeof(T) == 4) {
                v[i].x = fmaf(coef, z[0], v[i].x); v[i].y = fmaf(coef, z[1], v[i].y);
                v[i].z = fmaf(coef, z[2], v[i].z); v[i].w = fmaf(coef, z[3], v[i].w);
            } else {
                const float a0 = fmaf(coef, z[0], __uint_as_float(v[i].x << 16)), a1 = fmaf(coef, z[1], __uint_as_float(v[i].x & 0xFFFF0000u));
                const float a2 = fmaf(coef, z[2], __uint_as_float(v[i].y << 16)), a3 = fmaf(coef, z[3], __uint_as_float(v[i].y & 0xFFFF0000u));
                v[i] = make_uint2(pack_bf16x2(a0, a1), pack_bf16x2(a2, a3));
            }
            *reinterpret_cast<vec_t*>(pi) = v[i];
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (quad * 4 + c >= cols) break;
                if constexpr (sizeof(T) == 4) pi[c] = fmaf(coef, z[c], pi[c]);
                else pi[c] = f32_to_bf16(fmaf(coef, z[c], bf16_to_f32(pi[c])));
            }
        }
    }
}

template <typename T, bool VEC, int DENSE_ROWS>
static hipError_t launch_dense_rows(T* theta, int64_t rows, int64_t cols, int64_t ld, uint64_t seed, float scale, const double* g_dev, hipStream_t st) {
    const int64_t nquad = (cols + 3) / 4;
    const int64_t items = (rows + DENSE_ROWS - 1) / DENSE_ROWS * nquad;
    const dim3 grid((unsigned)((items + 255) / 256));
    hipLaunchKernelGGL((dense_axpy_kernel<T, VEC, DENSE_ROWS>), grid, dim3(256), 0, st, theta, rows, cols, ld, nquad, items,
                       (uint32_t)seed, (uint32_t)(seed >> 32), scale, g_dev);
    return hipGetLastError();
}
template <typename T>
static hipError_t launch_dense_typed(T* theta, int64_t rows, int64_t cols, int64_t ld, uint64_t seed, float scale, const double* g_dev, hipStream_t st) {
    if (cols % 4 == 0 && ld % 4 == 0 && reinterpret_cast<uintptr_t>(theta) % (4 * sizeof(T)) == 0)
        return launch_dense_rows<T, true, 2>(theta, rows, cols, ld, seed, scale, g_dev, st);
    if constexpr (sizeof(T) == 2)
        if ((double)rows * (double)cols >= 8e6) return launch_dense_rows<T, false, 2>(theta, rows, cols, ld, seed, scale, g_dev, st);
    return launch_dense_rows<T, false, 1>(theta, rows, cols, ld, seed, scale, g_dev, st);
}
hipError_t launch_dense_axpy(void* theta, int dtype, int64_t rows, int64_t cols, int64_t ld, uint64_t seed, float scale,
                             const double* g_dev, hipStream_t st) {
    if (rows == 0 || cols == 0) return hipSuccess;
    if (dtype == AGZO_BF16) return launch_dense_typed(static_cast<bf16_t*>(theta), rows, cols, ld, seed, scale, g_dev, st);
    return launch_dense_typed(static_cast<float*>(theta), rows, cols, ld, seed, scale, g_dev, st);
}

}  // namespace agzo
