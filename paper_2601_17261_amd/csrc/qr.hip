// Orthonormalisation steps of Alg. 1 ("[Q, ~] <- qr(Y)") for a tall d x r matrix, r <= 64:
// CholeskyQR2, everything past the fp32 input in fp64.  R from a Cholesky factor has a positive
// diagonal, which is the unique thin-QR factorisation of a full-rank Y.  A non-positive pivot
// (rank-deficient sketch) raises a device flag instead of producing NaNs.
//
// Three launches per QR (and one ahead of the second and third that sums many partials), coherence between them by kernel boundaries
// only (no device-scope fences):
//   1. gram        : Gram partials of Y per 128-row block (v_mfma_f64_16x16x4_f64)
//   2. apply_gram  : every block sums the partials in block order and factors the r x r matrix in LDS -> R1^-1;
//                    Q1 = Y R1^-1 (fp64, stored), then the Gram partials of Q1
//   3. apply_final : the same reduction and factorisation -> R2^-1; Q = Q1 R2^-1 (fp32), optionally
//                    also as three bf16 planes [3][rp][d]
// The orthonormalisations between power steps run a single pass (launches 1 and 3 only, launch 3 applying R1 to Y):
// Q1 = Q R2 with R2 upper triangular and positive on the diagonal, so the next sketch X^T X Q1 = (X^T X Q) R2 has
// the same thin-QR Q factor; the second pass only matters for the orthonormality of the basis that is returned.
// When the input arrives as per-token-range partial sketches, launch 1 sums them (fp64, fixed order)
// on the way in and stores the fp32 sketch, so no separate reduction kernel is needed.
//
// All of it is bound by chains of dependent steps.  The factorisation is blocked: one wave eliminates a 16 x 16 diagonal block
// in registers (its inverse along with it, no barrier), everything else - panels, trailing blocks, the inverse's other blocks,
// Y R^-1 - is 16 x 16 products on the fp64 matrix cores.  A column-by-column factorisation by the whole workgroup (two
// barriers a column) and a substitution with a thread per row took 159 us where this takes 42 (the single pass of seven 4B-sized
// layers, r = 64) and 10.9 where it takes 8.3 (0.6B-sized, r = 8); launch 1 at r = 64 65 and 22 us.
#include <type_traits>

#include "agzo_internal.h"

namespace agzo {

typedef double doublex4 __attribute__((ext_vector_type(4)));

constexpr int QR_ROWS = 128;   // rows per workgroup
constexpr int QR_LD = 17;      // row length of a 16 x 16 block in LDS (padded)
constexpr int QR_BLK = 16 * QR_LD;

template <int RP>
struct QrShape {
    static constexpr int NB = RP / 16, PAIRS = NB * (NB + 1) / 2;      // 16-column blocks; blocks of the upper triangle
    static constexpr int WAVES = NB == 1 ? 4 : 8, THREADS = 64 * WAVES;
    static constexpr int RB = QR_ROWS / 16 / WAVES;                     // 16-row blocks per wave
    static constexpr int LD = RP + 1;                                   // row length of the rows in LDS
    static constexpr size_t GRAM_SMEM = (size_t)QR_ROWS * LD * sizeof(float);
    static constexpr size_t FACTOR_SMEM = (size_t)2 * PAIRS * QR_BLK * sizeof(double);
    static constexpr size_t APPLY_GRAM_SMEM = FACTOR_SMEM + (size_t)QR_ROWS * LD * sizeof(double);
    static constexpr int PLANE_LD = QR_ROWS + 4;
    static constexpr size_t APPLY_FINAL_SMEM = FACTOR_SMEM + (size_t)RP * PLANE_LD * sizeof(float);
    // index of block (a, b), a <= b
    static __host__ __device__ constexpr int pair(int a, int b) { return a * NB - a * (a - 1) / 2 + (b - a); }
};

static inline int64_t qr_blocks(int64_t d) { return (d + QR_ROWS - 1) / QR_ROWS; }

size_t qr_workspace_bytes(int64_t d, int r) {
    const int rp = (r + 15) / 16 * 16;
    // [Q1 fp64 d*r][gram partials of Y and of Q1: up to nblk*rp*rp fp64 each]
    return (size_t)d * r * sizeof(double) + (size_t)2 * qr_blocks(d) * rp * rp * sizeof(double);
}

// ---- 16 x 16 products on the fp64 matrix cores.  Operand layout of v_mfma_f64_16x16x4_f64: lane l supplies element
// (l mod 16, k = l / 16) of both A and B; D (measured on gfx950): register i of lane l is row 4 i + l / 16, column l mod 16
// acc += A^T B (neg: -= ), A and B row-major blocks in LDS
__device__ __forceinline__ doublex4 mul_tn(const double* A, const double* B, doublex4 acc, bool neg) {
    const int lane = threadIdx.x & 63, at = (lane >> 4) * QR_LD + (lane & 15);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const double a = A[at + 4 * s * QR_LD];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(neg ? -a : a, B[at + 4 * s * QR_LD], acc, 0, 0, 0);
    }
    return acc;
}
// acc += A B
__device__ __forceinline__ doublex4 mul_nn(const double* A, const double* B, doublex4 acc, bool neg) {
    const int lane = threadIdx.x & 63, at = (lane >> 4) * QR_LD + (lane & 15), ta = (lane & 15) * QR_LD + (lane >> 4);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const double a = A[ta + 4 * s];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(neg ? -a : a, B[at + 4 * s * QR_LD], acc, 0, 0, 0);
    }
    return acc;
}
__device__ __forceinline__ doublex4 get_block(const double* G) {
    const int lane = threadIdx.x & 63;
    doublex4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = G[(4 * i + (lane >> 4)) * QR_LD + (lane & 15)];
    return v;
}
__device__ __forceinline__ void put_block(double* G, doublex4 v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 4; ++i) G[(4 * i + (lane >> 4)) * QR_LD + (lane & 15)] = v[i];
}

// ---- a wave eliminates one symmetric 16 x 16 block.  Lane (c, g) = (l mod 16, l / 16) holds rows 4 g .. 4 g + 3 of column c
// of the block and of the identity, which the same row operations turn into L^-1 (unit lower triangular; block = L D L^T)
// lane J of each 16 lanes, to all sixteen (row_newbcast)
template <int J>
__device__ __forceinline__ double row_bcast(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x150 + J, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x150 + J, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double read_lane(double x, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int J>
__device__ __forceinline__ void eliminate(double (&v)[4], double (&w)[4], int c, int g, int n, int& bad) {
    if constexpr (J < 16) {
        if (J > 0 && J % 4 == 0 && J >= n) return;               // (uniform) the rest is padding, which changes nothing
        constexpr int src = (J >> 2) * 16;                       // the lanes that hold row J
        double d = read_lane(v[J & 3], src + J);
        if (!(d > 0.0)) { bad |= 1 << J; d = 1.0; }
        double inv = __builtin_amdgcn_rcp(d);                    // hardware estimate, two Newton steps
        inv = fma(inv, fma(-d, inv, 1.0), inv);
        inv = fma(inv, fma(-d, inv, 1.0), inv);
        const double f = __shfl(v[J & 3], src + c) * inv, fw = __shfl(w[J & 3], src + c) * inv;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double col = row_bcast<J>(v[i]);                     // element (4 g + i, J)
            if (4 * g + i <= J) col = 0.0;
            v[i] = fma(-col, f, v[i]);
            w[i] = fma(-col, fw, w[i]);
        }
        eliminate<J + 1>(v, w, c, g, n, bad);
    }
}
// Rinv <- R^-1 of the block's factor R^T R (upper triangle, zeros below).  Rows and columns from n on are padding: unit diagonal.
// Returns nonzero (wave-uniform) on a non-positive pivot.  Sixteen columns are a chain of sixteen steps, so it ends behind the last four that are
// not all padding, the same bits: at rank 4 a factorisation takes 1.5 us less (a step of a 256-wide fp32 layer on 512 tokens 100.6 us with all steps and
// 93.7 so, of the 4B projections on 512 tokens 513 and 505), at rank 8 1 (of the 0.6B ones on 2048 365 and 360)
__device__ int factor16(const double* G, double* Rinv, int n) {
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    double v[4], w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 4 * g + i;
        w[i] = row == c ? 1.0 : 0.0;
        v[i] = (row < n && c < n) ? G[row * QR_LD + c] : w[i];
    }
    int bad = 0;
    eliminate<0>(v, w, c, g, n, bad);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 4 * g + i;
        double piv = __shfl(v[i], g * 16 + row);
        if ((bad >> row) & 1) piv = 1.0;
        // 1/sqrt(piv): hardware estimate refined by two Newton steps (full fp64 accuracy, no divide)
        double rs = __builtin_amdgcn_rsq(piv);
        rs = rs * fma(-0.5 * piv * rs, rs, 1.5);
        rs = rs * fma(-0.5 * piv * rs, rs, 1.5);
        Rinv[c * QR_LD + row] = c <= row ? w[i] * rs : 0.0;      // D^-1/2 L^-1, transposed
    }
    return bad;
}

// The workgroup turns the upper blocks of G = R^T R (LDS) into those of R^-1 (LDS), G's being overwritten.  Nonzero (the same
// in every thread) on a non-positive pivot
template <int RP>
__device__ int factor_inverse(double* G, double* Rinv, int r) {
    typedef QrShape<RP> Q;
    __shared__ int bad_s;
    const int tid = threadIdx.x, wave = tid >> 6;
    if (tid == 0) bad_s = 0;
    const doublex4 zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int p = 0; p < Q::NB; ++p) {
        __syncthreads();
        if (wave == 0) {
            const int bad = factor16(G + Q::pair(p, p) * QR_BLK, Rinv + Q::pair(p, p) * QR_BLK, min(16, r - 16 * p));
            if (bad && tid == 0) bad_s = 1;
        }
        __syncthreads();
        if (p + 1 < Q::NB) {
            const int q = p + 1 + wave;                          // panel: R_pq = R_pp^-T G_pq
            if (q < Q::NB) {
                double* blk = G + Q::pair(p, q) * QR_BLK;
                put_block(blk, mul_tn(Rinv + Q::pair(p, p) * QR_BLK, blk, zero, false));
            }
            __syncthreads();
            int job = 0;                                         // trailing blocks: G_ab -= R_pa^T R_pb
            for (int a = p + 1; a < Q::NB; ++a)
                for (int b = a; b < Q::NB; ++b, ++job) {
                    if (job % Q::WAVES != wave) continue;
                    double* blk = G + Q::pair(a, b) * QR_BLK;
                    put_block(blk, mul_tn(G + Q::pair(p, a) * QR_BLK, G + Q::pair(p, b) * QR_BLK, get_block(blk), true));
                }
        }
    }
#pragma unroll 1
    for (int dist = 1; dist < Q::NB; ++dist) {                   // R^-1_pq = -R^-1_pp sum over p < k <= q of R_pk R^-1_kq
        const int p = wave, q = p + dist;
        if (q < Q::NB) {
            doublex4 t = zero;
            for (int k = p + 1; k <= q; ++k) t = mul_nn(G + Q::pair(p, k) * QR_BLK, Rinv + Q::pair(k, q) * QR_BLK, t, false);
            double* blk = Rinv + Q::pair(p, q) * QR_BLK;
            put_block(blk, t);
            put_block(blk, mul_nn(Rinv + Q::pair(p, p) * QR_BLK, blk, zero, true));
        }
        __syncthreads();
    }
    return bad_s;
}

// Gram partial of the block's rows (LDS: Ys[row][LD], zero padded to QR_ROWS rows and RP columns; rows_pad: its rows up to a
// multiple of 4), written to
// partial[bx] as the 16 x 16 blocks of the upper triangle
template <int RP, typename T>
__device__ void gram_partial(const T* Ys, int rows_pad, double* partial, uint32_t bx) {
    typedef QrShape<RP> Q;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* out = partial + (int64_t)bx * Q::PAIRS * 256;
    if constexpr (Q::NB == 1) {
        // a single 16 x 16 block: the four waves split the rows (a lone wave would walk all of them through a chain
        // of dependent MFMAs) and their sums are added in wave order
        __shared__ double quarter[4][256];
        const int chunk = ((rows_pad / 4 + 3) / 4) * 4;               // rows per wave, a multiple of 4
        const int k_begin = min(wave * chunk, rows_pad), k_end = min(k_begin + chunk, rows_pad);
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int k0 = k_begin; k0 < k_end; k0 += 4) {
            const double a = (double)Ys[(k0 + (lane >> 4)) * Q::LD + (lane & 15)];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, acc, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) quarter[wave][(4 * i + (lane >> 4)) * 16 + (lane & 15)] = acc[i];
        __syncthreads();
        out[tid] = (quarter[0][tid] + quarter[1][tid]) + (quarter[2][tid] + quarter[3][tid]);
    } else {
        int job = 0;
        for (int a = 0; a < Q::NB; ++a)
            for (int b = a; b < Q::NB; ++b, ++job) {
                if (job % Q::WAVES != wave) continue;
                doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
                for (int k0 = 0; k0 < QR_ROWS; k0 += 4) {
                    const T* row = Ys + (k0 + (lane >> 4)) * Q::LD + (lane & 15);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)row[16 * a], (double)row[16 * b], acc, 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) out[Q::pair(a, b) * 256 + (4 * i + (lane >> 4)) * 16 + (lane & 15)] = acc[i];
            }
    }
}

struct QrSumDev { double* partial; int nblk; };

// Every block: sum over blocks of partial (block order, up to 32 loads of a thread in flight), then the workgroup factors
// it -> R^-1.  Block 0 reports a bad pivot.  smem: FACTOR_SMEM bytes; returns R^-1's blocks in it
template <int RP>
__device__ const double* reduce_and_factor(const double* partial, int nblk, double* smem, int r, int* flag, uint32_t bx) {
    typedef QrShape<RP> Q;
    constexpr int VEC = Q::NB == 1 ? 1 : 2, SIZE = Q::PAIRS * 256;
    typedef double vec_t __attribute__((ext_vector_type(VEC)));
    const int tid = threadIdx.x;
    for (int e = tid; e < SIZE / VEC; e += Q::THREADS) {
        vec_t sum = 0.0;
        const vec_t* src = reinterpret_cast<const vec_t*>(partial) + e;
        for (int b0 = 0; b0 < nblk; b0 += 32) {
            vec_t v[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) v[u] = (b0 + u < nblk) ? src[(int64_t)(b0 + u) * (SIZE / VEC)] : (vec_t)0.0;
#pragma unroll
            for (int u = 0; u < 32; ++u) sum += v[u];
        }
        const int at = e * VEC, blk = at >> 8, row = (at >> 4) & 15, col = at & 15;
        double* dst = smem + blk * QR_BLK + row * QR_LD + col;
#pragma unroll
        for (int i = 0; i < VEC; ++i) dst[i] = sum[i];
    }
    double* Rinv = smem + Q::PAIRS * QR_BLK;
    const int bad = factor_inverse<RP>(smem, Rinv, r);
    if (bad && tid == 0 && bx == 0) *flag = 1;
    if (Q::NB == 1) __syncthreads();
    return Rinv;
}

// The sum of reduce_and_factor() ahead of it, into the first block's partial: every block of the launches that follow reads all partials,
// and a compute unit takes in some 60 GB/s, so that 76 of 20 KB (r = 64, 9728 rows) are most of their time
template <int RP, int CAP>
__global__ __launch_bounds__(256) void qr_sum_kernel(const KBatch<QrSumDev, CAP> tb) {
    typedef QrShape<RP> Q;
    uint32_t bx, by;
    const QrSumDev& a = tb.a[kbatch_find(tb, bx, by)];
    double* at = a.partial + (int64_t)bx * 256 + threadIdx.x;
    double sum = 0.0;
    for (int b0 = 0; b0 < a.nblk; b0 += 32) {
        double v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) v[u] = b0 + u < a.nblk ? at[(int64_t)(b0 + u) * (Q::PAIRS * 256)] : 0.0;
#pragma unroll
        for (int u = 0; u < 32; ++u) sum += v[u];
    }
    *at = sum;
}

// the wave's rows of Y as operands (row l mod 16 of a 16-row block, columns l / 16 + 4 s of a column block), requested before
// the reduction and factorisation so that the memory latency runs under them
template <int RP, typename Tin>
__device__ __forceinline__ void load_rows(const Tin* __restrict__ Y, int64_t i0, int rows, int r, Tin (&y)[QrShape<RP>::RB][RP / 4]) {
    typedef QrShape<RP> Q;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int b = 0; b < Q::RB; ++b) {
        const int row = (wave * Q::RB + b) * 16 + (lane & 15);
#pragma unroll
        for (int s = 0; s < RP / 4; ++s) {
            const int col = 4 * s + (lane >> 4);
            y[b][s] = Y[(i0 + min(row, rows - 1)) * r + min(col, r - 1)];
        }
    }
#pragma unroll
    for (int b = 0; b < Q::RB; ++b)
#pragma unroll
        for (int s = 0; s < RP / 4; ++s)
            if ((wave * Q::RB + b) * 16 + (lane & 15) >= rows || 4 * s + (lane >> 4) >= r) y[b][s] = (Tin)0;
}
// column block q of a 16-row block of Y R^-1 (rows and columns as D lays them out)
template <int RP, typename Tin>
__device__ __forceinline__ doublex4 apply_rinv(const Tin (&y)[RP / 4], const double* Rinv, int q) {
    typedef QrShape<RP> Q;
    const int lane = threadIdx.x & 63, at = (lane >> 4) * QR_LD + (lane & 15);
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int p = 0; p < Q::NB; ++p) {
        if (p > q) break;
        const double* blk = Rinv + Q::pair(p, q) * QR_BLK + at;
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)y[4 * p + s], blk[4 * s * QR_LD], acc, 0, 0, 0);
    }
    return acc;
}

// per problem, what the launches of one factorisation need.  Input: S fp32 [d][r], or (splits != nullptr) partial sketches
// [nsplit][d][rp] ([nsplit][d] for r = 1) whose sum, rounded to fp32, is used for the factorisation and stored to S_out (not by qr1_small_kernel,
// behind which no launch reads it)
struct QrDev {
    const float* S; const float* splits; int nsplit; float* S_out; const float* Sin;
    int64_t d; int r; int nblk;
    double *Q1, *partial1, *partial2;
    float* Q; bf16_t* planes;
};

// launch 1
template <int RP, int CAP>
__global__ __launch_bounds__(QrShape<RP>::THREADS) void qr_gram_kernel(const KBatch<QrDev, CAP> tb) {
    typedef QrShape<RP> Q;
    extern __shared__ __align__(16) char qr_smem[];
    uint32_t bx, by;
    const QrDev& a = tb.a[kbatch_find(tb, bx, by)];
    float* Ys = reinterpret_cast<float*>(qr_smem);               // [QR_ROWS][LD]
    const int tid = threadIdx.x, r = a.r, nsplit = a.nsplit;
    const int64_t d = a.d, i0 = (int64_t)bx * QR_ROWS;
    const int rows = (int)min((int64_t)QR_ROWS, d - i0);
    const int rows_pad = (rows + 3) & ~3;
    if (a.splits != nullptr) {
        // sum of the partial sketches: a block's rows are one contiguous run of rows * rp floats in every split, so the
        // loads are plain 16-byte vectors, all splits of a vector in flight together (fp64 sum in split order)
        const int nvec = rows * RP / 4, total_vec = QR_ROWS * RP / 4;
        const float* base = a.splits + i0 * RP;
        float* S_out = a.S_out;
        auto finish = [&](int v, const double (&acc)[4]) {
            const int i = (v * 4) / RP, k0 = (v * 4) % RP;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float f = 0.f;
                if (v < nvec && k0 + c < r) {
                    f = (float)acc[c];
                    S_out[(i0 + i) * r + k0 + c] = f;
                }
                Ys[i * Q::LD + k0 + c] = f;
            }
        };
        // (at RP = 16 two vectors per thread, so that it has all its loads in flight at once: the kernel is bound by the
        // latency of these loads, the partials were written by the other XCDs)
        constexpr int VPT = Q::NB == 1 ? 2 : 1;
        for (int v0 = tid; v0 < total_vec; v0 += VPT * Q::THREADS) {
            double acc[VPT][4] = {};
            // N splits' loads at once; those past the last repeat it and are left out (never conditional: around a condition the
            // compiler waits for each load before the next, 14 us instead of 6 for seven 0.6B-sized layers)
            auto add = [&](auto NS) __attribute__((always_inline)) {
                constexpr int N = decltype(NS)::value;
                for (int sp0 = 0; sp0 < nsplit; sp0 += N) {
                    float4 x[VPT][N];
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        const float4* src = reinterpret_cast<const float4*>(base + (int64_t)min(sp0 + u, nsplit - 1) * d * RP);
#pragma unroll
                        for (int k = 0; k < VPT; ++k) x[k][u] = src[min(v0 + k * Q::THREADS, nvec - 1)];
                    }
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        const bool in = sp0 + u < nsplit;
#pragma unroll
                        for (int k = 0; k < VPT; ++k) {
                            acc[k][0] += in ? (double)x[k][u].x : 0.0; acc[k][1] += in ? (double)x[k][u].y : 0.0;
                            acc[k][2] += in ? (double)x[k][u].z : 0.0; acc[k][3] += in ? (double)x[k][u].w : 0.0;
                        }
                    }
                }
            };
            if (nsplit <= 8) add(std::integral_constant<int, 8>{});
            else add(std::integral_constant<int, 16>{});
#pragma unroll
            for (int k = 0; k < VPT; ++k)
                if (v0 + k * Q::THREADS < total_vec) finish(v0 + k * Q::THREADS, acc[k]);
        }
    } else {
        for (int e = tid; e < QR_ROWS * RP; e += Q::THREADS) {
            const int i = e / RP, k = e % RP;
            Ys[i * Q::LD + k] = (i < rows && k < r) ? a.S[(i0 + i) * r + k] : 0.f;
        }
    }
    __syncthreads();
    gram_partial<RP>(Ys, rows_pad, a.partial1, bx);
}

// launch 2: R1^-1 from the partials, Q1 = S R1^-1 for the block's rows (fp64, stored), Gram partials of Q1.
template <int RP, int CAP>
__global__ __launch_bounds__(QrShape<RP>::THREADS) void qr_apply_gram_kernel(const KBatch<QrDev, CAP> tb, int* flag) {
    typedef QrShape<RP> Q;
    extern __shared__ __align__(16) char qr_smem[];
    uint32_t bx, by;
    const QrDev& a = tb.a[kbatch_find(tb, bx, by)];
    double* Gs = reinterpret_cast<double*>(qr_smem);
    double* Ys = reinterpret_cast<double*>(qr_smem + Q::FACTOR_SMEM);      // [QR_ROWS][LD]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = a.r;
    const int64_t i0 = (int64_t)bx * QR_ROWS;
    const int rows = (int)min((int64_t)QR_ROWS, a.d - i0);
    float y[Q::RB][RP / 4];
    load_rows<RP>(a.Sin, i0, rows, r, y);
    const double* Rinv = reduce_and_factor<RP>(a.partial1, a.nblk, Gs, r, flag, bx);
#pragma unroll
    for (int b = 0; b < Q::RB; ++b)
#pragma unroll
        for (int q = 0; q < Q::NB; ++q) {
            const doublex4 v = apply_rinv<RP>(y[b], Rinv, q);
            const int col = 16 * q + (lane & 15);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = (wave * Q::RB + b) * 16 + 4 * i + (lane >> 4);
                Ys[row * Q::LD + col] = v[i];                              // (rows past the end, padding columns: zero)
                if (row < rows && col < r) a.Q1[(i0 + row) * r + col] = v[i];
            }
        }
    __syncthreads();
    gram_partial<RP>(Ys, (rows + 3) & ~3, a.partial2, bx);
}

// eight values of column c, rows i .. i + 7, as the planes [3][rp][d]
__device__ __forceinline__ void store_planes(const float* src, bf16_t* planes, int rp, int c, int64_t d, int64_t i) {
    uint32_t w[3][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        bf16_t h[2], m[2], l[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) split3_bf16(src[2 * u + k], h[k], m[k], l[k]);
        w[0][u] = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
        w[1][u] = (uint32_t)m[0] | ((uint32_t)m[1] << 16);
        w[2][u] = (uint32_t)l[0] | ((uint32_t)l[1] << 16);
    }
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint4*>(planes + ((int64_t)pl * rp + c) * d + i) = make_uint4(w[pl][0], w[pl][1], w[pl][2], w[pl][3]);
}

// launch 3: Q = Q1 R2^-1, rounded to fp32; planes (nullable, d % 8 == 0) receive the hi/mid/lo bf16 parts [3][rp][d].
// DOUBLE_IN: second pass of CholeskyQR2 (input Q1, partials of Q1); otherwise the single-pass form, Q = Y R1^-1 straight from
// launch 1's partials
template <int RP, bool DOUBLE_IN, int CAP>
__global__ __launch_bounds__(QrShape<RP>::THREADS) void qr_apply_final_kernel(const KBatch<QrDev, CAP> tb, int* flag) {
    typedef QrShape<RP> Q;
    extern __shared__ __align__(16) char qr_smem[];
    uint32_t bx, by;
    const QrDev& a = tb.a[kbatch_find(tb, bx, by)];
    double* Gs = reinterpret_cast<double*>(qr_smem);
    float* Qt = reinterpret_cast<float*>(qr_smem + Q::FACTOR_SMEM);        // [RP][PLANE_LD], transposed
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = a.r;
    const int64_t i0 = (int64_t)bx * QR_ROWS, d = a.d;
    const int rows = (int)min((int64_t)QR_ROWS, d - i0);
    typename std::conditional<DOUBLE_IN, double, float>::type y[Q::RB][RP / 4];
    if constexpr (DOUBLE_IN) load_rows<RP>(a.Q1, i0, rows, r, y);
    else load_rows<RP>(a.Sin, i0, rows, r, y);
    const double* Rinv = reduce_and_factor<RP>(DOUBLE_IN ? a.partial2 : a.partial1, a.nblk, Gs, r, flag, bx);
#pragma unroll
    for (int b = 0; b < Q::RB; ++b)
#pragma unroll
        for (int q = 0; q < Q::NB; ++q) {
            const doublex4 v = apply_rinv<RP>(y[b], Rinv, q);
            const int col = 16 * q + (lane & 15);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = (wave * Q::RB + b) * 16 + 4 * i + (lane >> 4);
                const float f = col < r ? (float)v[i] : 0.f;
                Qt[col * Q::PLANE_LD + row] = f;
                if (row < rows && col < r) a.Q[(i0 + row) * r + col] = f;
            }
        }
    if (a.planes == nullptr) return;
    __syncthreads();
    // eight rows of one column and plane per thread and pass: 16-byte stores
    for (int e = tid; e < RP * (QR_ROWS / 8); e += Q::THREADS) {
        const int i = (e % (QR_ROWS / 8)) * 8, c = e / (QR_ROWS / 8);
        if (i < rows) store_planes(Qt + c * Q::PLANE_LD + i, a.planes, RP, c, d, i0 + i);
    }
}

// ---- up to 512 rows and 16 columns: the launches above as one workgroup.  Bound by the latency of a launch each, they took 4.6 + 6.3 us
// (single pass of 256 rows) and 4.6 + 7.5 + 6.2; this takes some 7.5 and 11 (r = 16; 6 and 10 for four columns), 2 of it for a factorisation.  Everything is added in the order of those launches, so the results are the same bits and a
// call may take either way.  (A wave has 64 rows, two quarters of a Gram partial there: with all four in a row the matrix instructions took
// a third of the time, and more rows than these take longer than the launches.)
constexpr int QRS_BLOCKS = 4, QRS_WAVES = 2 * QRS_BLOCKS, QRS_ROWS = QRS_BLOCKS * QR_ROWS, QRS_LD = 17;
constexpr size_t qrs_smem(int blocks) { return (size_t)blocks * QR_ROWS * QRS_LD * sizeof(double) + (4 * QRS_BLOCKS * 256 + 2 * QR_BLK) * sizeof(double); }
template <int CAP>
__global__ __launch_bounds__(64 * QRS_WAVES) void qr_small_kernel(const KBatch<QrDev, CAP> tb, int refine, int* flag) {
    extern __shared__ __align__(16) char qr_smem[];
    const QrDev& a = tb.a[CAP == 1 ? 0 : blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lc = lane & 15, lg = lane >> 4;
    const int r = a.r, d = (int)a.d, nblk = a.nblk, nsplit = a.nsplit;
    double* parts = reinterpret_cast<double*>(qr_smem);                   // [blocks][4][256]
    double *G = parts + 4 * QRS_BLOCKS * 256, *Rinv = G + QR_BLK;
    char* rows_at = reinterpret_cast<char*>(Rinv + QR_BLK);               // rows in fp32, then in fp64, then Q transposed
    float* Ys = reinterpret_cast<float*>(rows_at);
    // (loads are never conditional on the lane: around a condition the compiler waits for each before the next)
    if (a.splits != nullptr) {
        const int nvec = d * 4, total = nblk * QR_ROWS * 4;
        for (int v0 = tid; v0 < total; v0 += 2 * 64 * QRS_WAVES) {
            double acc[2][4] = {};
            for (int sp0 = 0; sp0 < nsplit; sp0 += 8) {
                float4 x[2][8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        x[k][u] = reinterpret_cast<const float4*>(a.splits + (int64_t)min(sp0 + u, nsplit - 1) * d * 16)[min(v0 + k * 64 * QRS_WAVES, nvec - 1)];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool in = sp0 + u < nsplit;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        acc[k][0] += in ? (double)x[k][u].x : 0.0; acc[k][1] += in ? (double)x[k][u].y : 0.0;
                        acc[k][2] += in ? (double)x[k][u].z : 0.0; acc[k][3] += in ? (double)x[k][u].w : 0.0;
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int v = v0 + k * 64 * QRS_WAVES, i = v >> 2, k0 = (v & 3) * 4;
                if (v >= total) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool in = v < nvec && k0 + c < r;
                    const float f = in ? (float)acc[k][c] : 0.f;
                    if (in) a.S_out[(int64_t)i * r + k0 + c] = f;
                    Ys[i * QRS_LD + k0 + c] = f;
                }
            }
        }
    } else {
        const int total = nblk * QR_ROWS * 16;                            // (four to a thread at least)
        for (int e0 = tid; e0 < total; e0 += 4 * 64 * QRS_WAVES) {
            float x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * 64 * QRS_WAVES;
                x[u] = a.S[(int64_t)min(e >> 4, d - 1) * r + min(e & 15, r - 1)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * 64 * QRS_WAVES;
                if (e < total) Ys[(e >> 4) * QRS_LD + (e & 15)] = ((e >> 4) < d && (e & 15) < r) ? x[u] : 0.f;
            }
        }
    }
    __syncthreads();
    const int block = wave >> 1, half = wave & 1, row0 = block * QR_ROWS;
    // the Gram matrix of the rows and R^-1: a wave's four quarters side by side, then the waves' sums
    auto gram_factor = [&](const auto* Y) __attribute__((always_inline)) {
        if (block < nblk) {
            const int rows_pad = (min(QR_ROWS, d - row0) + 3) & ~3, chunk = ((rows_pad / 4 + 3) / 4) * 4;
            doublex4 acc[2] = {};
            for (int t = 0; t < chunk; t += 4)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int at = (2 * half + q) * chunk + t;
                    if (at < rows_pad) {
                        const double y = (double)Y[(row0 + at + lg) * QRS_LD + lc];
                        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(y, y, acc[q], 0, 0, 0);
                    }
                }
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) parts[(block * 4 + 2 * half + q) * 256 + (4 * i + lg) * 16 + lc] = acc[q][i];
        }
        __syncthreads();
        if (tid < 256) {
            double sum = 0.0;
            for (int b = 0; b < nblk; ++b) {
                const double* p = parts + b * 4 * 256 + tid;
                sum += (p[0] + p[256]) + (p[512] + p[768]);
            }
            G[(tid >> 4) * QR_LD + (tid & 15)] = sum;
        }
        if (factor_inverse<16>(G, Rinv, r) && tid == 0) *flag = 1;
        __syncthreads();
    };
    constexpr int RB = QR_ROWS / 32;                                      // 16-row blocks of a wave
    const int rw = row0 + half * (QR_ROWS / 2);
    doublex4 v[RB];
    auto apply = [&](const auto* Y) __attribute__((always_inline)) {
        if (block < nblk) {
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                typename std::remove_const<typename std::remove_reference<decltype(*Y)>::type>::type y[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) y[s] = Y[(rw + b * 16 + lc) * QRS_LD + 4 * s + lg];
                v[b] = apply_rinv<16>(y, Rinv, 0);
            }
        }
        __syncthreads();                                                  // what follows goes where the rows are
    };
    gram_factor(Ys);
    apply(Ys);
    if (refine) {
        double* Y1 = reinterpret_cast<double*>(rows_at);
        if (block < nblk)
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) Y1[(rw + b * 16 + 4 * i + lg) * QRS_LD + lc] = v[b][i];
        __syncthreads();
        gram_factor(Y1);
        apply(Y1);
    }
    const int ld = nblk * QR_ROWS + 4;
    float* Qt = reinterpret_cast<float*>(rows_at);                        // [16][ld]
    if (block < nblk)
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = rw + b * 16 + 4 * i + lg;
                const float f = lc < r ? (float)v[b][i] : 0.f;
                Qt[lc * ld + row] = f;
                if (row < d && lc < r) a.Q[(int64_t)row * r + lc] = f;
            }
    if (a.planes == nullptr) return;
    __syncthreads();
    for (int e = tid; e < 16 * nblk * (QR_ROWS / 8); e += 64 * QRS_WAVES) {
        const int i = (e % (nblk * (QR_ROWS / 8))) * 8, c = e / (nblk * (QR_ROWS / 8));
        if (i < d) store_planes(Qt + c * ld + i, a.planes, 16, c, a.d, i);
    }
}

// ---- r = 1 (the paper's operating point): the thin QR of a single column with a positive diagonal is the column
// divided by its norm, so the orthonormalisation is a sum of squares and a scaling: two small launches, no Gram
// matrix, no factorisation, and nothing for a second pass to refine.
constexpr int QR1_ROWS = 256;    // rows per workgroup, one per thread: the chain of loads is what takes the time

// launch 1: y_i = the column (or the fp64 sum of its partial sketches in split order, rounded to fp32 and stored to
// S_out like the general path does), partial[b] = sum of y_i^2 over the block's rows (fp64, fixed order)
template <int CAP>
__global__ __launch_bounds__(256) void qr1_sumsq_kernel(const KBatch<QrDev, CAP> tb) {
    __shared__ double red[4];
    uint32_t bx, by;
    const QrDev& a = tb.a[kbatch_find(tb, bx, by)];
    const int tid = threadIdx.x;
    const int64_t i = (int64_t)bx * QR1_ROWS + tid;
    float y = 0.f;
    if (i < a.d) {
        if (a.splits != nullptr) {
            double acc = 0.0;
            for (int sp0 = 0; sp0 < a.nsplit; sp0 += 16) {
                float x[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) x[u] = sp0 + u < a.nsplit ? a.splits[(int64_t)(sp0 + u) * a.d + i] : 0.f;
#pragma unroll
                for (int u = 0; u < 16; ++u) acc += (double)x[u];
            }
            y = (float)acc;
            a.S_out[i] = y;
        } else {
            y = a.S[i];
        }
    }
    double ss = (double)y * (double)y;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    if (tid == 0) a.partial1[bx] = (red[0] + red[1]) + (red[2] + red[3]);
}

// launch 2: q = y / sqrt(sum of the partials) -> Q fp32 [d][1] and, if asked, the bf16 planes [3][rp][d] (rows of the
// padding columns zero; d % 8 == 0).  A sum that is not positive (an all-zero sketch) raises the numeric flag.
template <int CAP>
__global__ __launch_bounds__(256) void qr1_scale_kernel(const KBatch<QrDev, CAP> tb, int rp, int* flag) {
    uint32_t bx, by;
    const QrDev& a = tb.a[kbatch_find(tb, bx, by)];
    const int tid = threadIdx.x;
    const int64_t i0 = (int64_t)bx * QR1_ROWS, i = i0 + tid;
    const float y = i < a.d ? a.Sin[i] : 0.f;
    double sum = 0.0;
    for (int b0 = 0; b0 < a.nblk; b0 += 16) {                  // uniform: every thread adds the same values
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = b0 + u < a.nblk ? a.partial1[b0 + u] : 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) sum += v[u];
    }
    if (!(sum > 0.0)) {
        if (tid == 0 && bx == 0) *flag = 1;
        sum = 1.0;
    }
    const float q = (float)((double)y * (1.0 / sqrt(sum)));
    if (i < a.d) a.Q[i] = q;
    if (a.planes == nullptr) return;
    if (i < a.d) {
        bf16_t part[3];
        split3_bf16(q, part[0], part[1], part[2]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) a.planes[(int64_t)pl * rp * a.d + i] = part[pl];
    }
    const int rest = rp - 1;
    for (int e = tid; e < 3 * rest * (QR1_ROWS / 8); e += 256) {
        const int64_t col = i0 + (e % (QR1_ROWS / 8)) * 8;
        const int row = e / (QR1_ROWS / 8), pl = row / rest;
        if (col < a.d) *reinterpret_cast<uint4*>(a.planes + ((int64_t)pl * rp + 1 + row - pl * rest) * a.d + col) = make_uint4(0, 0, 0, 0);
    }
}
int qr_norm_blocks(int64_t d) { return (int)((d + QR1_ROWS - 1) / QR1_ROWS); }

// Both launches as one workgroup a column, for columns that nobody else has to read in between: the sums in the same order, so the same bits.
// The last launch of a lone layer's basis: 37.4 us with the two and 36.6 so at 1024 wide on 128 tokens, 41.4 and 40.7 at 256 on 2048.  1536 wide it is the
// same and 2048 wide 1 to 3 % slower (1000 tokens: 48.3 and 49.8), so a row a thread is the most it takes
constexpr int QR1S_ROWS = 1024;
template <int CAP>
__global__ __launch_bounds__(QR1S_ROWS) void qr1_small_kernel(const KBatch<QrDev, CAP> tb, int rp, int* flag) {
    __shared__ double red[QR1S_ROWS / 64];
    const QrDev& a = tb.a[CAP == 1 ? 0 : blockIdx.x];
    const int i = threadIdx.x, d = (int)a.d, nsplit = a.nsplit, at = min(i, d - 1);
    float y;
    if (a.splits != nullptr) {
        double acc = 0.0;
        for (int sp0 = 0; sp0 < nsplit; sp0 += 16) {
            float x[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) x[u] = sp0 + u < nsplit ? a.splits[(int64_t)(sp0 + u) * d + at] : 0.f;
#pragma unroll
            for (int u = 0; u < 16; ++u) acc += (double)x[u];
        }
        y = (float)acc;
    } else {
        y = a.S[at];
    }
    if (i >= d) y = 0.f;
    double ss = (double)y * (double)y;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    if ((i & 63) == 0) red[i >> 6] = ss;
    __syncthreads();
    double sum = 0.0;
    for (int b = 0; b < a.nblk; ++b) sum += (red[4 * b] + red[4 * b + 1]) + (red[4 * b + 2] + red[4 * b + 3]);
    if (!(sum > 0.0)) {
        if (i == 0) *flag = 1;
        sum = 1.0;
    }
    const double scale = 1.0 / sqrt(sum);
    const float q = (float)((double)y * scale);
    if (i < d) a.Q[i] = q;
    if (a.planes == nullptr) return;
    if (i < d) {
        bf16_t part[3];
        split3_bf16(q, part[0], part[1], part[2]);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) a.planes[(int64_t)pl * rp * d + i] = part[pl];
    }
    const int rest = rp - 1;                                   // the padding columns: zero
    for (int row = 0; row < 3 * rest; ++row) {
        const int pl = row / rest;
        if (i < d) a.planes[((int64_t)pl * rp + 1 + row - pl * rest) * d + i] = 0;
    }
}
template <int CAP>
static bool qr1_small(const KBatch<QrDev, CAP>& tb, const KBatch<QrDev, CAP>& scaled) {
    for (int m = 0; m < tb.n; ++m)
        if (tb.a[m].d > QR1S_ROWS) return false;
    return scaled.n == tb.n;
}

// tb: every column; scaled: those that this factorisation normalises itself
template <int CAP>
static hipError_t launch_qr1(const KBatch<QrDev, CAP>& tb, unsigned blocks, const KBatch<QrDev, CAP>& scaled, unsigned scaled_blocks, int rp, int* flag,
                             bool refine, hipStream_t st) {
    if (refine && qr1_small(tb, scaled)) {
        hipLaunchKernelGGL(qr1_small_kernel<CAP>, dim3((unsigned)tb.n), dim3(QR1S_ROWS), 0, st, tb, rp, flag);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(qr1_sumsq_kernel<CAP>, dim3(blocks), dim3(256), 0, st, tb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || scaled_blocks == 0) return e;      // the launch below consumes what this one would have written
    hipLaunchKernelGGL(qr1_scale_kernel<CAP>, dim3(scaled_blocks), dim3(256), 0, st, scaled, rp, flag);
    return hipGetLastError();
}

// Bytes of Gram partials from which on they are summed ahead.  agzo_qr, us, summed by every block and ahead: r = 64, 2048 rows (320 KB) 64.5
// and 65.6, 2560 (400 KB) 66.1 and 65.9, 4096 (640 KB) 71 and 67, 9728 (1.5 MB) 90 and 72; r = 32, 9728 (456 KB) 37.8 and 37.2; r = 16, 40000
// (626 KB) 58 and 50.  The single pass of seven 4B-sized layers, r = 64: 41 and 30 + 5.7.  A step of them on 128 tokens, r = 26 (456 KB):
// 438 and 445, 8B-sized (576 KB), before there were sums ahead and now: 695 and 684
constexpr int64_t kSumAhead = 512 * 1024;
template <int RP, int CAP>
static hipError_t launch_qr_rp(const KBatch<QrDev, CAP>& tb, unsigned blocks, int* flag, bool refine, hipStream_t st) {
    typedef QrShape<RP> Q;
    static bool attr_set = false;
    if (!attr_set) {
        const auto allow = [](const void* f, size_t bytes) { return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes); };
        hipError_t e = allow(reinterpret_cast<const void*>(qr_gram_kernel<RP, CAP>), Q::GRAM_SMEM);
        if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(qr_apply_gram_kernel<RP, CAP>), Q::APPLY_GRAM_SMEM);
        if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(qr_apply_final_kernel<RP, true, CAP>), Q::APPLY_FINAL_SMEM);
        if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(qr_apply_final_kernel<RP, false, CAP>), Q::APPLY_FINAL_SMEM);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const dim3 grid(blocks), block(Q::THREADS);
    // the partials summed ahead where a block would read many bytes of them
    int64_t most = 0;
    for (int m = 0; m < tb.n; ++m) most = tb.a[m].nblk > most ? tb.a[m].nblk : most;
    const bool ahead = most * Q::PAIRS * 2048 > kSumAhead;
    KBatch<QrDev, CAP> one = tb;                  // what the launches behind the sums take
    for (int m = 0; ahead && m < one.n; ++m) one.a[m].nblk = 1;
    auto sums = [&](bool second) -> hipError_t {
        if (!ahead) return hipSuccess;
        KBatch<QrSumDev, CAP> su;
        su.n = tb.n;
        for (int m = 0; m < tb.n; ++m) {
            su.first[m] = (uint32_t)(m * Q::PAIRS);
            su.gx[m] = Q::PAIRS;
            su.a[m] = QrSumDev{second ? tb.a[m].partial2 : tb.a[m].partial1, tb.a[m].nblk};
        }
        hipLaunchKernelGGL((qr_sum_kernel<RP, CAP>), dim3((unsigned)(tb.n * Q::PAIRS)), dim3(256), 0, st, su);
        return hipGetLastError();
    };
    hipLaunchKernelGGL((qr_gram_kernel<RP, CAP>), grid, block, Q::GRAM_SMEM, st, tb);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = sums(false);
    if (e != hipSuccess) return e;
    if (!refine) {
        hipLaunchKernelGGL((qr_apply_final_kernel<RP, false, CAP>), grid, block, Q::APPLY_FINAL_SMEM, st, one, flag);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((qr_apply_gram_kernel<RP, CAP>), grid, block, Q::APPLY_GRAM_SMEM, st, one, flag);
    e = hipGetLastError();
    if (e == hipSuccess) e = sums(true);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((qr_apply_final_kernel<RP, true, CAP>), grid, block, Q::APPLY_FINAL_SMEM, st, one, flag);
    return hipGetLastError();
}

// Whether one workgroup a problem does it: few rows, fewer where partial sketches are to be summed.  agzo_qr, us, three launches and one: 100
// rows 15.4 and 10.6, 256 16.9 and 11.7, 384 17.1 and 13.8, 512 17.2 and 14.7, 1024 17.8 and 21.  A step of one layer: fp32, 256 wide on
// 512 tokens 117 and 106, 512 on 300 142 and 137; bf16, 256 wide on 300 tokens 118 and 108, on 8000 (16 partial sketches) 216 and 207, but
// 504 on 512 (4) 135 and 141
template <int CAP>
static bool qr_small(const KBatch<QrDev, CAP>& tb) {
    for (int m = 0; m < tb.n; ++m)
        if (tb.a[m].d > (tb.a[m].splits ? QRS_ROWS / 2 : QRS_ROWS)) return false;
    return true;
}
template <int CAP>
static hipError_t launch_qr_small(const KBatch<QrDev, CAP>& tb, int* flag, bool refine, hipStream_t st) {
    static bool attr_set = false;
    if (!attr_set) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(qr_small_kernel<CAP>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)qrs_smem(QRS_BLOCKS));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    int most = 0;
    for (int m = 0; m < tb.n; ++m) most = tb.a[m].nblk > most ? tb.a[m].nblk : most;
    hipLaunchKernelGGL(qr_small_kernel<CAP>, dim3((unsigned)tb.n), dim3(64 * QRS_WAVES), qrs_smem(most), st, tb, refine ? 1 : 0, flag);
    return hipGetLastError();
}

template <int CAP>
static hipError_t launch_qr_cap(const KBatch<QrDev, CAP>& tb, unsigned blocks, int rp, int* flag, bool refine, hipStream_t st) {
    if (rp == 16 && qr_small(tb)) return launch_qr_small(tb, flag, refine, st);
    switch (rp) {
        case 16: return launch_qr_rp<16>(tb, blocks, flag, refine, st);
        case 32: return launch_qr_rp<32>(tb, blocks, flag, refine, st);
        case 48: return launch_qr_rp<48>(tb, blocks, flag, refine, st);
        case 64: return launch_qr_rp<64>(tb, blocks, flag, refine, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_qr_many(const QrArgs* a, int n, int* numeric_flag, bool refine, hipStream_t st) {
    if (n < 0 || n > kBatchMax) return hipErrorInvalidValue;
    KBatch<QrDev> tb, scaled;
    tb.n = scaled.n = 0;
    uint64_t blocks = 0, scaled_blocks = 0;
    int rp = 0, rank1 = -1;
    for (int m = 0; m < n; ++m) {
        if (a[m].d == 0) continue;
        if (rp == 0) rp = a[m].rp;
        if (rank1 < 0) rank1 = (a[m].r == 1);
        // one padded rank per launch, and single columns (normalised, not factored) apart from the others
        if (a[m].rp != rp || (a[m].r == 1) != (rank1 == 1) || (a[m].defer && a[m].r != 1)) return hipErrorInvalidValue;
        QrDev q;
        q.S = a[m].S; q.splits = a[m].splits; q.nsplit = a[m].nsplit; q.S_out = a[m].S_out;
        q.Sin = a[m].splits ? a[m].S_out : a[m].S;
        q.d = a[m].d; q.r = a[m].r; q.nblk = (int)qr_blocks(a[m].d);
        // (the partials first: their vectors are aligned whatever d and r are)
        q.partial1 = reinterpret_cast<double*>(a[m].workspace);
        q.partial2 = q.partial1 + (size_t)q.nblk * rp * rp;
        q.Q1 = q.partial2 + (size_t)q.nblk * rp * rp;
        q.Q = a[m].Q; q.planes = a[m].planes;
        if (rank1 == 1) q.nblk = qr_norm_blocks(a[m].d);        // (partials: fewer than those reserved)
        if (rank1 == 1 && !a[m].defer) {
            scaled.first[scaled.n] = (uint32_t)scaled_blocks; scaled.gx[scaled.n] = (uint32_t)q.nblk; scaled.a[scaled.n++] = q;
            scaled_blocks += (uint64_t)q.nblk;
        }
        tb.first[tb.n] = (uint32_t)blocks; tb.gx[tb.n] = (uint32_t)q.nblk; tb.a[tb.n++] = q;
        blocks += (uint64_t)q.nblk;
    }
    if (tb.n == 0) return hipSuccess;
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (rank1 == 1) {
        if (tb.n == 1) {
            KBatch<QrDev, 1> one = kbatch_one(tb), none = one;
            none.n = scaled.n;
            return launch_qr1(one, (unsigned)blocks, none, (unsigned)scaled_blocks, rp, numeric_flag, refine, st);
        }
        return launch_qr1(tb, (unsigned)blocks, scaled, (unsigned)scaled_blocks, rp, numeric_flag, refine, st);
    }
    if (tb.n == 1) return launch_qr_cap(kbatch_one(tb), (unsigned)blocks, rp, numeric_flag, refine, st);
    return launch_qr_cap(tb, (unsigned)blocks, rp, numeric_flag, refine, st);
}

hipError_t launch_qr(const float* S, const float* splits, int nsplit, int rp, float* S_out, int64_t d, int r, float* Q,
                     bf16_t* planes, void* workspace, int* numeric_flag, bool refine, hipStream_t st) {
    const QrArgs a{S, splits, nsplit, rp, S_out, d, r, Q, planes, workspace};
    return launch_qr_many(&a, 1, numeric_flag, refine, st);
}

}  // namespace agzo
